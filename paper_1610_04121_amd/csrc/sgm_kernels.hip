// Single-pair SGM kernels for gfx950 and their host-side launchers.  The
// stage bodies live in sgm_device.h; each kernel here maps its grid onto one
// stereo pair.
#include <algorithm>
#include <hip/hip_runtime.h>

#include <cstdlib>

#include "sgm_agg.h"
#include "sgm_device.h"
#include "sgm_plan.h"
#include "sgm_row.h"

namespace sgm {

namespace {

using namespace dev;

__global__ __launch_bounds__(256) void census97_kernel(CensusArgs a) { census97_block(a, blockIdx.x, blockIdx.y, blockIdx.z); }

__global__ __launch_bounds__(256) void census_generic_kernel(CensusArgs a, int rx, int ry) {
    census_generic_block(a, rx, ry, blockIdx.x, blockIdx.y, blockIdx.z);
}

__global__ __launch_bounds__(256) void census_cost_kernel(CensusCostArgs a) {
    extern __shared__ __align__(16) uint8_t cc_smem[];
    census_cost_block(a, blockIdx.x, blockIdx.y, cc_smem);
}

template <bool RB, int DP, int RUN, int AUX>
__global__ __launch_bounds__(kCostThreads) void cost_kernel(CostArgs a) {
    using U = CostUnit<DP, RUN>;
    __shared__ uint64_t words[kCostThreads / 64][U::words];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nx = (a.W + U::PX - 1) / U::PX;
    const int unit = blockIdx.x * (kCostThreads / 64) + wave;
    if (unit < nx * a.H) cost_unit<RB, DP, RUN, AUX>(a, unit % nx, unit / nx, threadIdx.x & 63, words[wave]);
}

template <bool RB, int RUN, int AUX>
void launch_cost_t(const CostArgs& a, hipStream_t stream) {
    const int px = cost_unit_px(a.Dp, RUN), units = (a.W + px - 1) / px * a.H, per = kCostThreads / 64;
    auto k = a.Dp == 64 ? cost_kernel<RB, 64, RUN, AUX> : a.Dp == 128 ? cost_kernel<RB, 128, RUN, AUX> : cost_kernel<RB, 256, RUN, AUX>;
    hipLaunchKernelGGL(k, dim3((units + per - 1) / per), dim3(kCostThreads), 0, stream, a);
}

template <typename LT, bool NT, bool FOLD>
__global__ __launch_bounds__(1024) void wta_kernel(WtaArgs a) {
    extern __shared__ uint32_t wta_smem[];
    wta_row<LT, NT, FOLD>(a, blockIdx.x, wta_smem);
}

// Winner-take-all of two SGMs in one launch (full left-right check): rows
// 0 .. H-1 of the left-base sums give D_L, blocks H .. 2H-1 the rows of the
// right-base sums, D_R.
template <typename LT, bool NT, bool FOLD>
__global__ __launch_bounds__(1024) void wta_pair_kernel(WtaArgs l, WtaArgs r) {
    extern __shared__ uint32_t wta_smem[];
    const int y = blockIdx.x;
    if (y < l.H)
        wta_row<LT, NT, FOLD>(l, y, wta_smem);
    else
        wta_row<LT, NT, FOLD>(r, y - l.H, wta_smem);
}

// The final pass (see final_pass_block): NPL = n_paths - 1 stored planes;
// NT: non-temporal plane loads.
template <int Dp, int NPL, bool NT>
__global__ __launch_bounds__(kFinalThreads) void final_pass_kernel(FinalArgs f) {
    extern __shared__ __align__(16) uint8_t fp_smem[];
    final_pass_block<Dp, NPL, NT>(f, blockIdx.x, fp_smem);
}

__global__ __launch_bounds__(256) void post_kernel(PostArgs a) {
    extern __shared__ uint16_t post_smem[];
    post_row(a, blockIdx.x, post_smem);
}

// Debug tap: S = sum of L_r over planes (of L_r - C; of L_r without cost),
// u16 [H][W][D].  Plane `skip` (-1: none) is left out.
template <typename LT>
__global__ void sum_planes_kernel(const void* lbuf, const uint8_t* cost, size_t plane, uint16_t* s, int W, int H, int D,
                                  int Dp, int nplanes, int skip) {
    const size_t n = (size_t)W * H * D;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const size_t p = i / D, d = i - p * D;
        uint32_t acc = 0;
        for (int k = 0; k < nplanes; ++k)
            if (k != skip) acc += reinterpret_cast<const LT*>(lbuf)[plane * k + p * Dp + d] + (cost ? cost[p * Dp + d] : 0);
        s[i] = (uint16_t)acc;
    }
}

// Debug tap: one L_r (a plane of L_r - C and the costs, or a plane of L_r or
// the cost volume alone) as u16 [H][W][D].
template <typename LT>
__global__ void extract_plane_kernel(const LT* src, const uint8_t* cost, uint16_t* out, int W, int H, int D, int Dp) {
    const size_t n = (size_t)W * H * D;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const size_t p = i / D, d = i - p * D;
        out[i] = (uint16_t)(src[p * Dp + d] + (cost ? cost[p * Dp + d] : 0));
    }
}

}  // namespace

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
bool plan_finish(Plan& p, const char** why) {
    auto fail = [&](const char* m) {
        if (why) *why = m;
        return false;
    };
    if (p.W < 1 || p.H < 1) return fail("width and height must be >= 1");
    if (p.W > kMaxWidth) return fail("width must be <= 16000");
    if (p.D < 1 || p.D > kMaxDisp) return fail("max_disp must be in [1, 256]");
    if (!(p.n_paths == 2 || p.n_paths == 4 || p.n_paths == 8)) return fail("n_paths must be 2, 4 or 8");
    if (p.cw < 1 || p.ch < 1 || !(p.cw & 1) || !(p.ch & 1)) return fail("census window sides must be odd and >= 1");
    if (p.cw > 31 || p.ch > 15) return fail("census window must be at most 31 wide and 15 tall");
    if (!p.csct && p.cw * p.ch > 64) return fail("full census window must have <= 64 pixels");
    if (p.csct && (p.cw * p.ch - 1) / 2 > 64) return fail("CSCT window must have <= 64 pairs");
    if (p.P1 < 0 || p.P2 < 0) return fail("P1 and P2 must be >= 0");
    if (p.P1 > 65535) return fail("P1 must be <= 65535");
    p.cmax = p.csct ? (p.cw * p.ch - 1) / 2 : p.cw * p.ch - 1;
    // the largest penalty of one step bounds L_r <= Cmax + penalty: P2, or
    // with adaptive P2 (max(P1, P2 / (1 + g)) per step) the larger of P1, P2
    const long long pmax = p.adaptive ? std::max(p.P1, p.P2) : p.P2;
    if ((long long)p.n_paths * (p.cmax + pmax) > 65535)
        return fail(p.adaptive ? "n_paths * (Cmax + max(P1, P2)) must be <= 65535 (16-bit summed costs, adaptive P2)"
                               : "n_paths * (Cmax + P2) must be <= 65535 (16-bit summed costs)");
    if (p.lr_thr < 0) return fail("lr threshold must be >= 0");
    p.Dp = padded_disp(p.D);
    p.pmax = (int)pmax;
    // the planes hold L_r - C in [0, pmax] (from the last term of Eq. 3)
    p.l16 = pmax > 255;
    p.wide = p.cmax + pmax > 255;
    // Normal stores leave a frame's planes in the 256 MiB memory-side cache
    // for the row kernel (or WTA) to read back.  When the planes and the cost volume
    // do not fit, the dirty planes would be written back while the WTA reads,
    // so they are stored non-temporally instead.  (The count is of whole planes
    // in every direction, also for frames that keep checkpoints of the
    // horizontal ones and move less.)
    {
        const long long cells = (long long)p.W * p.H * p.Dp;
        const long long nsgm = p.lr_full ? 2 : 1;
        const long long bytes = nsgm * cells * (p.n_paths * (p.l16 ? 2 : 1) + 1);
        p.nt_store = bytes > kMallBytes;
    }
    // one L_r plane (u16) must stay below 2 GiB: kernels address planes with
    // 32-bit byte offsets
    if ((long long)p.W * p.H * p.Dp > (1LL << 30)) return fail("width * height * padded disparities must be <= 2^30");
    return true;
}

static size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

size_t workspace_bytes(const Plan& p) {
    const size_t npx = (size_t)p.W * p.H;
    const size_t cells = npx * p.Dp;
    const int nsgm = p.lr_full ? 2 : 1;
    return align256(cells) + align256(cells * nsgm * p.n_paths * (p.l16 || p.wide ? 2 : 1)) + 2 * align256(npx * 2) +
           2 * align256(8 * (npx + kCensusGuard)) + align256(4 * (size_t)p.H) + (p.lr_full ? align256(cells) : 0);
}

Workspace workspace_carve(const Plan& p, void* base) {
    const size_t npx = (size_t)p.W * p.H;
    const size_t cells = npx * p.Dp;
    uint8_t* b = static_cast<uint8_t*>(base);
    Workspace ws;
    ws.cost = b;
    b += align256(cells);
    ws.lbuf = b;
    b += align256(cells * (p.lr_full ? 2 : 1) * p.n_paths * (p.l16 || p.wide ? 2 : 1));
    ws.dl = reinterpret_cast<uint16_t*>(b);
    b += align256(npx * 2);
    ws.dr = reinterpret_cast<uint16_t*>(b);
    b += align256(npx * 2);
    ws.census_l = reinterpret_cast<uint64_t*>(b) + kCensusGuard;
    b += align256(8 * (npx + kCensusGuard));
    ws.census_r = reinterpret_cast<uint64_t*>(b) + kCensusGuard;
    b += align256(8 * (npx + kCensusGuard));
    ws.rowcnt = reinterpret_cast<int*>(b);
    b += align256(4 * (size_t)p.H);
    if (p.lr_full) ws.cost_r = b;
    return ws;
}

static hipError_t launch_census_pair(const Plan& p, const uint8_t* left, const uint8_t* right, uint64_t* cl,
                                     uint64_t* cr, int nimg, hipStream_t stream, int* zero = nullptr) {
    CensusArgs a{{left, right}, {cl, cr}, p.W, p.H, p.csct ? 1 : 0, zero, zero ? p.H : 0};
    if (p.cw == 9 && p.ch == 7) {
        dim3 grid((p.W + kCenTX - 1) / kCenTX, (p.H + kCenTY - 1) / kCenTY, nimg);
        hipLaunchKernelGGL(census97_kernel, grid, dim3(256), 0, stream, a);
    } else {
        dim3 grid((p.W + 15) / 16, (p.H + 15) / 16, nimg);
        hipLaunchKernelGGL(census_generic_kernel, grid, dim3(256), 0, stream, a, (p.cw - 1) / 2, (p.ch - 1) / 2);
    }
    return hipGetLastError();
}

hipError_t launch_census(const Plan& p, const Workspace& ws, const uint8_t* left, const uint8_t* right,
                         hipStream_t stream) {
    return launch_census_pair(p, left, right, ws.census_l, ws.census_r, 2, stream, ws.rowcnt);
}

bool census_cost_fusable(const Plan& p) { return p.cc_fused && p.cw == 9 && p.ch == 7; }

hipError_t launch_matching_cost(const Plan& p, const Workspace& ws, const uint8_t* left, const uint8_t* right,
                                bool need_cost, hipStream_t stream) {
    if (p.lr_full) {  // census words, then both cost volumes
        hipError_t e = launch_census(p, ws, left, right, stream);
        if (e == hipSuccess) e = launch_cost(p, ws, stream, false);
        if (e == hipSuccess) e = launch_cost(p, ws, stream, true);
        return e;
    }
    const bool fusable = census_cost_fusable(p);
    hipError_t e = hipSuccess;
    if (need_cost && fusable) {
        const CcLayout L = cc_layout(p.D, p.Dp);
        CensusCostArgs a{left, right, ws.cost, p.W, p.H, p.D, p.Dp, p.cmax, p.csct ? 1 : 0, ws.rowcnt, p.H};
        hipLaunchKernelGGL(census_cost_kernel, dim3((p.W + kCcTX - 1) / kCcTX, p.H), dim3(256), L.bytes, stream, a);
        e = hipGetLastError();
    }
    // census words in global memory: for the fused aggregation, and for the
    // cost kernel of windows other than 9x7
    if (e == hipSuccess && (fused_aggregation(p) || (need_cost && !fusable)))
        e = launch_census(p, ws, left, right, stream);
    if (e == hipSuccess && need_cost && !fusable) e = launch_cost(p, ws, stream);
    return e;
}

hipError_t launch_cost(const Plan& p, const Workspace& ws, hipStream_t stream, bool right_base) {
    if (right_base && !ws.cost_r) return hipErrorInvalidValue;
    const CostArgs a = right_base ? CostArgs{ws.census_r, ws.census_l, ws.cost_r, p.W, p.H, p.D, p.Dp, p.cmax}
                                  : CostArgs{ws.census_l, ws.census_r, ws.cost, p.W, p.H, p.D, p.Dp, p.cmax};
    // Pixels per lane: 8; 2 where 8 leave at most one wavefront per SIMD, so
    // that the launch is a shorter chain (96x64, D = 32: 3.2 and 4.3 us).  With
    // every SIMD busy the staging of the match words counts (1600x1200,
    // D = 128: 8 pixels 42 us, 4 45, 2 65).
    const int px = cost_unit_px(p.Dp, 8);
    const bool few = (long long)((p.W + px - 1) / px) * p.H <= 1024;
    // A volume larger than the memory-side cache is written past it: the
    // aggregation cannot find it there (1920x1080, D = 256, 531 MB: 88 us, with
    // sc1 108); smaller ones stay (1280x720, D = 64: sc1 13.8 us, 17.4).
    const bool nt = (long long)(p.lr_full ? 2 : 1) * p.W * p.H * p.Dp > kMallBytes;
    if (right_base)
        few  ? launch_cost_t<true, 2, kStoreSc1>(a, stream)
        : nt ? launch_cost_t<true, 8, kStoreNT>(a, stream)
             : launch_cost_t<true, 8, kStoreSc1>(a, stream);
    else
        few  ? launch_cost_t<false, 2, kStoreSc1>(a, stream)
        : nt ? launch_cost_t<false, 8, kStoreNT>(a, stream)
             : launch_cost_t<false, 8, kStoreSc1>(a, stream);
    return hipGetLastError();
}

static void fill_agg_args(const Plan& p, const Workspace& ws, const uint8_t* left, const uint8_t* right, int SH,
                          int SV, AggArgs& a, bool skip_last) {
    a.base = SliceArgs{ws.cost, ws.census_l, ws.census_r, nullptr, (uint32_t)((size_t)p.W * p.H * p.Dp),
                       p.W, p.H, p.D, p.P1, p.P2, p.cmax, 0, 0};
    a.lbuf = ws.lbuf;
    // directions of the left-base SGM (planes 0 .. P-1) and, for the full
    // left-right check, of the right-base SGM (planes P .. 2P-1)
    const int nsgm = p.lr_full ? 2 : 1;
    const int all = nsgm * p.n_paths;
    const int last = skip_last ? last_direction(p) : -1;
    a.ndirs = all - (skip_last ? 1 : 0);
    // longest slices first, so that they start first
    int order[kMaxLaunchDirs], n = 0;
    const bool horiz_first = p.W >= p.H;
    for (int pass = 0; pass < 2; ++pass)
        for (int i = 0; i < all; ++i) {
            if (i == last) continue;
            const bool horiz = direction(p.n_paths, i % p.n_paths).ry == 0;
            if ((horiz == horiz_first) == (pass == 0)) order[n++] = i;
        }
    int acc = 0;
    for (int k = 0; k < a.ndirs; ++k) {
        const Dir d = direction(p.n_paths, order[k] % p.n_paths);
        const int S = d.ry == 0 ? SH : SV;
        a.rx[k] = d.rx;
        a.ry[k] = d.ry;
        // without the last direction the stored planes close up
        a.plane_index[k] = order[k] - (last >= 0 && order[k] > last ? 1 : 0);
        a.cost[k] = order[k] < p.n_paths ? ws.cost : ws.cost_r;
        a.img[k] = order[k] < p.n_paths ? left : right;
        a.start[k] = acc;
        acc += (slice_count(p.W, p.H, d) + S - 1) / S;
    }
    a.start[a.ndirs] = acc;
    a.total = acc;
    for (int k = 0; k < a.ndirs; ++k) {
        a.paired[k] = 0;
        if (k + 1 < a.ndirs && !(k > 0 && a.paired[k - 1]) && a.rx[k] == -a.rx[k + 1] && a.ry[k] == -a.ry[k + 1] &&
            (a.rx[k] == 0 || a.ry[k] == 0) && order[k] / p.n_paths == order[k + 1] / p.n_paths &&
            a.start[k + 1] - a.start[k] == a.start[k + 2] - a.start[k + 1])
            a.paired[k] = 1;
    }
}

// Group widths (lanes per slice).  More lanes make a step shorter and the
// wavefronts more.  With at most one wavefront per SIMD (1024) the longest
// chain sets the time, so the widest shape that fits one round wins; beyond
// that, what counts is how full the last round is.  Whole calls (us), median +
// check: 451x377, D = 128, 8 paths: 16/16 (865 wavefronts) 98, 32/16 (1054)
// 110; 451x377, D = 128, 4 paths: 32/32 (828) 69.5, 32/16 75.3; 640x480, D =
// 128, 4 paths: 32/16 (800) 95, 32/32 (1120) 108; 640x480, D = 256, 2 paths:
// 64/32 (800) 112, 32/16 135; 640x480, D = 128, 8 paths: 64/16 (1920, 0.94 of
// two rounds) 155, 32/16 (1440, 0.70) 161; 800x600, D = 128, 8 paths: 32/32
// (3000, 0.98) 255, 32/16 (1800, 0.88) 272; 1242x375, D = 128, 8 paths: 64/16
// (2613, 0.85) 248, 32/16 (2238, 0.73) 262; D = 256: 1000x600, 4 paths 16/16
// (800) 300, 32/16 (1100) 330, 32/32 (1600) 307; 1080x720 346, 374, 356; 600x800
// 251, 284, 256; 1242x375, 4 paths 32/16 (998) 253, 16/16 267; 1242x375, 8 paths
// 64/16 446, 32/16 470, 16/16 516.  With 64 levels a 16-lane step is
// as short as a 32-lane one (320x240: 43.2 and 45.0), except with many
// directions over several rounds (1242x375, 8 paths: 32/16 151, 16/16 159).
// 64 horizontal lanes beyond one round only pay with diagonals (640x480 4
// paths: 115).  Two SGMs (the full check) are not narrowed to fit one round
// (1242x375, 4 paths: 16/16 239, 32/16 223).
void default_lanes(const Plan& p, int* gh, int* gv) {
    constexpr int kSimds = 1024;
    const int nsgm = p.lr_full ? 2 : 1;
    const int horiz = p.n_paths == 2 ? 1 : 2, other = p.n_paths - horiz;
    auto waves = [&](int h, int v) {
        const int sh = 64 / h, sv = 64 / v;
        return nsgm * (horiz * ((p.H + sh - 1) / sh) + other * ((p.W + sv - 1) / sv));
    };
    auto set = [&](int h, int v) {
        *gh = h;
        *gv = v;
    };
    // a step that computes its costs loads a census word per level of a lane:
    // the fewest levels (256 levels, 4 paths: 640x480 256 us, 32/16 508; 1000x600
    // 563, 16/16 1084, 32/16 983; 16-bit planes 808, 1726 and 1450)
    if (p.Dp == 256 && fused_aggregation(p)) return set(64, 32);
    if (p.Dp == 64) {
        const bool many = waves(16, 16) > kSimds && nsgm * p.n_paths >= 8;
        return many ? set(32, 16) : set(16, 16);
    }
    if (p.Dp == 256 && waves(64, 32) <= kSimds) return set(64, 32);
    if (waves(32, 32) <= kSimds) return set(32, 32);
    if (waves(32, 16) <= kSimds) return set(32, 16);
    if (waves(16, 16) <= kSimds && nsgm == 1) return set(16, 16);
    auto fill = [&](int h, int v) {  // share of the rounds' SIMDs in use
        const int w = waves(h, v);
        return (double)w / (kSimds * (double)((w + kSimds - 1) / kSimds));
    };
    set(32, 16);
    const int shapes[3][2] = {{16, 16}, {32, 32}, {64, 16}};
    for (const auto& sh : shapes)
        if ((sh[0] < 64 || p.n_paths == 8) && fill(sh[0], sh[1]) > 1.05 * fill(*gh, *gv)) set(sh[0], sh[1]);
}

// Wavefronts per slice (dev::Split).  Splitting divides the dependent chain
// and costs the steps until the segments' values meet, so it pays where the
// longest chain takes well over the time of the launch's bytes.  Estimates: a
// step 45 ns + 6 per level of a lane (72 ns at 4, 93 at 8), bytes at 6.3 TB/s.
// Whole calls, unsplit and split (us): 320x240, D = 64, 4 paths (chain over
// bytes 3.6) 44.0, 35.2 in 4; 1280x720, D = 64, 4 paths (1.6) 155, 140 in 2;
// 1242x375, D = 128, 4 paths (1.5) 160, 138 in 2; 640x480, D = 128, 2 paths
// (2.4) 85, 77 in 2, 78 in 4; but 800x600, D = 128, 4 paths (1.0) 136, 143;
// with 256 levels 320x240, 4 paths (1.3) 60, 68 and 640x480, 2 paths (1.3)
// 114, 126.  With 8 paths the wavefronts fill the device (160x120, D = 128:
// 37, 43), and short slices do not repay the rounds (96x64, D = 128: 25.0,
// 26.4).  On unrelated images, where the values never meet, the rounds take
// the time the split saves and more: 640x480, D = 128, 2 paths 101 (flat
// images 85); so 2 paths, whose chain is the shorter one, split in 2 at most.
static int slice_segments(const Plan& p, int gh, int gv, bool checkpoints) {
    if (p.l16 || fused_aggregation(p) || p.n_paths == 8 || std::max(p.W, p.H) < 160) return 1;
    auto chain_ns = [&](int steps, int lanes) { return steps * (45.0 + 6.0 * (p.Dp / lanes)); };
    const double chain = std::max(chain_ns(p.W, gh), chain_ns(p.H, gv));
    const int horiz = p.n_paths == 2 ? 1 : 2, stored = checkpoints ? p.n_paths - horiz : p.n_paths;
    const double bytes = (p.lr_full ? 2.0 : 1.0) * p.W * p.H * p.Dp * (p.n_paths + stored + (checkpoints ? 0.1 : 0.0));
    const double ratio = chain / (bytes / 6300.0);  // 6.3 TB/s = 6300 bytes per ns
    if (ratio < (p.Dp == 256 ? 1.5 : 1.4)) return 1;
    return ratio > 2.3 && p.n_paths == 4 ? 4 : 2;
}

// It stores L_r itself, which byte planes hold up to Cmax + pmax = 255; past
// that, up to pmax = 255, the stored-cost aggregation on byte planes of L - C
// takes its place, which is 2 to 7 times as fast as this one on 16-bit planes
// (P2 = 220: 640x480, D = 128, 4 paths 96 us and 222; 320x240, D = 256 60 and 275).
bool fused_aggregation(const Plan& p) { return p.fused && !p.lr_full && !p.adaptive && (p.l16 || !p.wide); }

hipError_t launch_aggregate(const Plan& p, const Workspace& ws, hipStream_t stream, const uint8_t* left,
                            const uint8_t* right, bool skip_last, bool checkpoints) {
    int gh = p.lanes_h, gv = p.lanes_v;
    if (gh <= 0 || gv <= 0) default_lanes(p, &gh, &gv);
    if (p.Dp == 64) gh = std::min(gh, 32);  // 64 lanes need at least 2 levels per lane
    if (p.adaptive && (!left || (p.lr_full && !right))) return hipErrorInvalidValue;
    AggArgs a;
    fill_agg_args(p, ws, left, right, 64 / gh, 64 / gv, a, skip_last);
    a.ckpt = checkpoints ? 1 : 0;
    a.gh = gh;
    a.gv = gv;
    a.split = slice_segments(p, gh, gv, checkpoints);
    // the store policy is an instruction operand: a second instantiation of
    // the plain (stored-cost, constant-P2) kernels
    const AggVariant v{p.l16, fused_aggregation(p), p.adaptive, p.nt_store && !p.adaptive && !fused_aggregation(p)};
    if (p.Dp == 64) return launch_agg_64(a, v, stream);
    if (p.Dp == 128) return launch_agg_128(a, v, stream);
    return launch_agg_256(a, v, stream);
}

// Not past Cmax + pmax = 255: byte planes of L - C hold more, but the plain
// route, which such frames always took, is faster (640x480, 4 paths, P2 = 250:
// D = 64 64 us against 111, D = 128 95 against 139).
bool final_pass_active(const Plan& p) {
    if (!p.final_pass || p.wide || p.lr_full || p.adaptive || fused_aggregation(p)) return false;
    return final_smem_bytes(p.Dp, p.W, p.lrcheck) <= 64 * 1024;
}

template <int Dp, int NPL>
static hipError_t launch_final_t(const Plan& p, const FinalArgs& f, hipStream_t stream) {
    using L = FinalLayout<Dp>;
    const size_t smem = final_smem_bytes(Dp, p.W, p.lrcheck);
    auto k = p.nt_store ? final_pass_kernel<Dp, NPL, true> : final_pass_kernel<Dp, NPL, false>;
    hipLaunchKernelGGL(k, dim3((p.H + L::R - 1) / L::R), dim3(kFinalThreads), smem, stream, f);
    return hipGetLastError();
}

template <int Dp>
static hipError_t launch_final_d(const Plan& p, const FinalArgs& f, hipStream_t stream) {
    switch (p.n_paths) {
        case 2: return launch_final_t<Dp, 1>(p, f, stream);
        case 4: return launch_final_t<Dp, 3>(p, f, stream);
        default: return launch_final_t<Dp, 7>(p, f, stream);
    }
}

hipError_t launch_final_pass(const Plan& p, const Workspace& ws, uint16_t* out, hipStream_t stream, uint16_t* s_out) {
    if (!final_pass_active(p)) return hipErrorInvalidValue;
    const Dir d = direction(p.n_paths, last_direction(p));
    const bool post = p.median || p.lrcheck;
    const size_t plane = (size_t)p.W * p.H * p.Dp;
    FinalArgs f;
    f.agg = SliceArgs{ws.cost, ws.census_l, ws.census_r, nullptr, (uint32_t)plane, p.W, p.H, p.D, p.P1, p.P2,
                      p.cmax, d.rx, d.ry};
    f.planes = static_cast<const uint8_t*>(ws.lbuf);
    f.plane = plane;
    f.wta = WtaArgs{nullptr, plane, post ? ws.dl : out, p.lrcheck ? ws.dr : nullptr, p.W, p.H, p.D, p.Dp,
                    p.n_paths - 1, p.subpixel ? 1 : 0};
    f.s_out = s_out;
    if (p.Dp == 64) return launch_final_d<64>(p, f, stream);
    if (p.Dp == 128) return launch_final_d<128>(p, f, stream);
    return launch_final_d<256>(p, f, stream);
}

bool post_folded(const Plan& p) { return p.post_in_wta && (p.median || p.lrcheck) && !final_pass_active(p); }

hipError_t launch_aggregate_wta(const Plan& p, const Workspace& ws, const uint8_t* left, const uint8_t* right,
                                uint16_t* out, hipStream_t stream, hipEvent_t mid_event, bool post_in_wta) {
    const bool fp = final_pass_active(p), row = row_kernel_active(p, post_in_wta);
    hipError_t e = launch_aggregate(p, ws, stream, left, right, fp, row);
    if (e == hipSuccess && mid_event) e = hipEventRecord(mid_event, stream);
    if (e == hipSuccess)
        e = fp ? launch_final_pass(p, ws, out, stream)
               : (row ? launch_row(p, ws, left, right, out, stream) : launch_wta(p, ws, out, stream, post_in_wta));
    return e;
}

// The row kernel trades two plane passes for running the horizontal
// directions twice, so it pays where the planes' bytes set the time.  The
// whole call with plain WTA against row kernel (us, one frame): 320x240 D = 64
// 4 paths (19.7 M cell-paths) 44.6 / 44.4, 320x240 D = 128 8 paths (79 M) 59.8 /
// 60.7, 451x377 D = 128 2 paths (44 M) 68.2 / 69.8, 640x480 D = 64 4 paths
// (79 M) 79.3 / 76.7, 640x480 D = 128 4 paths (157 M) 99.8 / 94.8, 1280x720
// D = 128 8 paths (944 M) 491 / 421; 96x64 D = 64 4 paths (1.6 M) 24.0 / 25.6.
constexpr long long kRowKernelCells = 72ll << 20;

bool row_kernel_active(const Plan& p, bool post_in_wta) {
    return (long long)p.W * p.H * p.Dp * p.n_paths > kRowKernelCells && !final_pass_active(p) && !fused_aggregation(p) &&
           !post_in_wta;
}

// Whether the L_r planes were stored non-temporally, so the WTA streams them
// the same way: the plain aggregation kernels follow p.nt_store; the
// adaptive-P2 and census-computing ones always store them normally.
static bool planes_nt(const Plan& p) { return p.nt_store && !p.adaptive && !fused_aggregation(p); }

static PostArgs post_args(const Plan& p, const Workspace& ws, uint16_t* out) {
    return PostArgs{ws.dl, ws.dr, out, p.W, p.H, p.median ? 1 : 0, p.lrcheck ? 1 : 0, p.lr_thr, p.subpixel ? 1 : 0};
}

hipError_t launch_row(const Plan& p, const Workspace& ws, const uint8_t* left, const uint8_t* right, uint16_t* out,
                      hipStream_t stream) {
    const bool post = p.median || p.lrcheck;
    const size_t plane = (size_t)p.W * p.H * p.Dp;
    RowLaunch a{};
    a.l = RowArgs{ws.cost, ws.lbuf, left, post ? ws.dl : out, p.lrcheck && !p.lr_full ? ws.dr : nullptr,
                  p.W, p.H, p.D, p.P1, p.P2, p.n_paths, p.adaptive ? 1 : 0, p.subpixel ? 1 : 0};
    if (p.lr_full) {  // the right-base SGM's winners are D_R
        a.r = a.l;
        a.r.cost = ws.cost_r;
        a.r.planes = static_cast<const uint8_t*>(ws.lbuf) + plane * p.n_paths * (p.l16 ? 2 : 1);
        a.r.img = right;
        a.r.dl = ws.dr;
        a.r.subpixel = 0;
    }
    const RowVariant v{p.n_paths, p.l16, planes_nt(p), 2 * p.pmax <= 255, p.subpixel};
    const int blocks = p.lr_full ? 2 * p.H : p.H;
    const size_t smem = row_smem_bytes(p.W, a.l.dr != nullptr);
    auto launch = p.Dp == 64 ? launch_row_64 : (p.Dp == 128 ? launch_row_128 : launch_row_256);
    return launch(a, v, blocks, row_waves(p.W, p.Dp, p.l16), smem, stream);
}

hipError_t launch_wta(const Plan& p, const Workspace& ws, uint16_t* out, hipStream_t stream, bool post_in_wta) {
    // Without the post stage inside, frames come here up to kRowKernelCells
    // cell-paths, whose planes and costs (at most 3/2 a byte plane's cells, 5/2
    // a 16-bit one's, with 2 paths) are stored non-temporally only for two SGMs
    // on 16-bit planes, or with the census-computing aggregation, whose never are.
    static_assert(2 * 3 * kRowKernelCells / 2 <= kMallBytes && 5 * kRowKernelCells / 2 <= kMallBytes, "unreached variants");
    const bool nt = planes_nt(p);
    const bool post = p.median || p.lrcheck;
    const bool fold = post_in_wta && post;
    const uint8_t* cost = fused_aggregation(p) ? nullptr : ws.cost;  // planes of L - C need C
    if (fold && !ws.rowcnt) return hipErrorInvalidValue;
    if (p.lr_full) {
        const size_t plane = (size_t)p.W * p.H * p.Dp;
        const void* rbuf = static_cast<const uint8_t*>(ws.lbuf) + plane * p.n_paths * (p.l16 ? 2 : 1);
        WtaArgs l{ws.lbuf, plane, ws.dl, nullptr, p.W, p.H, p.D, p.Dp, p.n_paths, p.subpixel ? 1 : 0, cost};
        WtaArgs r{rbuf, plane, ws.dr, nullptr, p.W, p.H, p.D, p.Dp, p.n_paths, 0, ws.cost_r};
        size_t smem = 0;
        if (fold) {  // D_L and D_R rows come from separate blocks
            for (WtaArgs* w : {&l, &r}) {
                w->rowcnt = ws.rowcnt;
                w->contrib = 2;
                w->post = post_args(p, ws, out);
            }
            smem = 2 * (size_t)p.W;  // the post stage's D_R medians
        }
        auto k = fold ? (p.l16 ? (nt ? wta_pair_kernel<uint16_t, true, true> : wta_pair_kernel<uint16_t, false, true>)
                               : (nt ? wta_pair_kernel<uint8_t, true, true> : wta_pair_kernel<uint8_t, false, true>))
                      : (p.l16 ? (nt ? wta_pair_kernel<uint16_t, true, false> : wta_pair_kernel<uint16_t, false, false>)
                               : wta_pair_kernel<uint8_t, false, false>);
        hipLaunchKernelGGL(k, dim3(2 * p.H), dim3(1024), smem, stream, l, r);
        return hipGetLastError();
    }
    WtaArgs a{ws.lbuf, (size_t)p.W * p.H * p.Dp, post ? ws.dl : out, p.lrcheck ? ws.dr : nullptr,
              p.W, p.H, p.D, p.Dp, p.n_paths, p.subpixel ? 1 : 0, cost};
    if (fold) {
        a.rowcnt = ws.rowcnt;
        a.post = post_args(p, ws, out);
    }
    // the right-view keys; with the post stage inside, its D_R medians reuse them
    const size_t smem = p.lrcheck ? 4 * (size_t)(p.W + kWtaGuard) : 0;
    // the planes are read the way they were stored: non-temporally when they
    // exceed the memory-side cache and the aggregation stored them so
    auto k = fold ? (p.l16 ? (nt ? wta_kernel<uint16_t, true, true> : wta_kernel<uint16_t, false, true>)
                           : (nt ? wta_kernel<uint8_t, true, true> : wta_kernel<uint8_t, false, true>))
                  : (p.l16 ? wta_kernel<uint16_t, false, false> : wta_kernel<uint8_t, false, false>);
    hipLaunchKernelGGL(k, dim3(p.H), dim3(1024), smem, stream, a);
    return hipGetLastError();
}

hipError_t launch_post(const Plan& p, const Workspace& ws, uint16_t* out, hipStream_t stream) {
    if (!p.median && !p.lrcheck) return hipSuccess;  // the WTA wrote `out`
    const PostArgs a = post_args(p, ws, out);
    hipLaunchKernelGGL(post_kernel, dim3(p.H), dim3(256), p.lrcheck ? 2 * (size_t)p.W : 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_pipeline(const Plan& p, const Workspace& ws, const uint8_t* left,
                           const uint8_t* right, uint16_t* out, hipStream_t stream, hipEvent_t* events) {
    hipError_t e = hipSuccess;
    auto mark = [&](int i) {
        if (events && e == hipSuccess) e = hipEventRecord(events[i], stream);
    };
    mark(0);
    if (e == hipSuccess) e = launch_matching_cost(p, ws, left, right, !fused_aggregation(p), stream);
    mark(1);
    const bool fold = post_folded(p);
    if (e == hipSuccess)
        e = launch_aggregate_wta(p, ws, left, right, out, stream, events ? events[2] : nullptr, fold);
    mark(3);
    if (e == hipSuccess && !fold) e = launch_post(p, ws, out, stream);
    mark(4);
    return e;
}

hipError_t launch_census_only(const Plan& p, const uint8_t* img, uint64_t* out, hipStream_t stream) {
    return launch_census_pair(p, img, img, out, out, 1, stream);
}

hipError_t launch_sum_planes(const Plan& p, const Workspace& ws, uint16_t* s_out, hipStream_t stream, int skip,
                             int nplanes) {
    const size_t plane = (size_t)p.W * p.H * p.Dp;
    if (nplanes < 0) nplanes = p.n_paths;
    const uint8_t* cost = fused_aggregation(p) ? nullptr : ws.cost;
    if (p.l16)
        hipLaunchKernelGGL(sum_planes_kernel<uint16_t>, dim3(1024), dim3(256), 0, stream, ws.lbuf, cost, plane, s_out,
                           p.W, p.H, p.D, p.Dp, nplanes, skip);
    else
        hipLaunchKernelGGL(sum_planes_kernel<uint8_t>, dim3(1024), dim3(256), 0, stream, ws.lbuf, cost, plane, s_out,
                           p.W, p.H, p.D, p.Dp, nplanes, skip);
    return hipGetLastError();
}

hipError_t launch_extract_plane(const Plan& p, const Workspace& ws, int plane, uint16_t* out,
                                hipStream_t stream) {
    const size_t cells = (size_t)p.W * p.H * p.Dp;
    const uint8_t* cost = fused_aggregation(p) ? nullptr : (plane < p.n_paths ? ws.cost : ws.cost_r);
    const uint8_t* none = nullptr;
    if (plane < 0)  // -1: the cost volume, -2: the right-base cost volume
        hipLaunchKernelGGL(extract_plane_kernel<uint8_t>, dim3(1024), dim3(256), 0, stream,
                           plane == -2 ? ws.cost_r : ws.cost, none, out, p.W, p.H, p.D, p.Dp);
    else if (p.l16)
        hipLaunchKernelGGL(extract_plane_kernel<uint16_t>, dim3(1024), dim3(256), 0, stream,
                           reinterpret_cast<const uint16_t*>(ws.lbuf) + cells * plane, cost, out, p.W, p.H, p.D, p.Dp);
    else
        hipLaunchKernelGGL(extract_plane_kernel<uint8_t>, dim3(1024), dim3(256), 0, stream,
                           reinterpret_cast<const uint8_t*>(ws.lbuf) + cells * plane, cost, out, p.W, p.H, p.D, p.Dp);
    return hipGetLastError();
}

}  // namespace sgm
