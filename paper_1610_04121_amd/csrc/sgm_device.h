// Device code of the SGM pipeline for gfx950 (CDNA4, 64-wide wavefronts),
// shared by the single-pair kernels and the batched kernels.  Each stage is
// a device function that takes its block coordinates explicitly.
//
// Stages (Sec. 2 of arXiv 1610.04121):
//   census97_block / census_generic_block  census words (Eq. 1 / full window)
//   cost_block      Hamming cost volume C (Eq. 2), u8
//   aggregate_wave  Eq. 3 along one direction, one group of lanes per slice
//   wta_row         S = sum_r L_r and winner-take-all (Eq. 4), right view
//   post_row        3x3 median and left-right consistency check
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "sgm_common.h"

namespace sgm {
namespace dev {



// The byte the cost volume holds at padded levels d >= D.  The aggregation
// on byte planes reads it as the high byte of 0x03FF (unpack_selector).
constexpr uint32_t kPadCost = 3;

__device__ inline int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// 16-byte store at byte offset `ofs` of [base, base + bytes) through a
// range-checked buffer resource, with device scope (sc1) or non-temporal:
// measured faster than plain stores for the cost volume (640x480, D = 128:
// sc1 12.1 us, plain 15.5; 1920x1080, D = 256: 115, 116, non-temporal 93).
constexpr int kStoreNT = 2, kStoreSc1 = 16;
template <int AUX = kStoreSc1>
__device__ inline void store16(void* base, uint32_t bytes, uint32_t ofs, uint4 v) {
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(base, 0, (int)bytes, 0x00020000);
    __builtin_amdgcn_raw_buffer_store_b128((unsigned __attribute__((ext_vector_type(4)))){v.x, v.y, v.z, v.w}, r, ofs,
                                           0, AUX);
}

// ---------------------------------------------------------------------------
// Census kernel: 9x7 windows (full or center-symmetric), register blocked.
// A block covers 64 x 16 pixels of one image (blockIdx.z); each thread makes
// 4 consecutive census words of one row.  The block stages a (16 + 6) x 72
// tile (clamp-to-edge), and each thread reads its 12 x 7 window patch as
// 3 aligned dwords per row.  The comparisons s(u, v) = [u >= v] of the 4
// pixels run byte-parallel in one dword (census_words4).
// ---------------------------------------------------------------------------
constexpr int kCenTX = 64, kCenTY = 16;

struct CensusArgs {
    const uint8_t* img[2];
    uint64_t* out[2];
    int W, H, csct;
    // block (0, 0, 0) clears zero[0 .. nzero) for the frame's later launches
    // (the row counters of the post stage inside the WTA launch)
    int* zero = nullptr;
    int nzero = 0;
};

__device__ inline void census_clear(const CensusArgs& a, int bx, int by, int z) {
    if (a.zero && (bx | by | z) == 0)
        for (int i = threadIdx.x; i < a.nzero; i += blockDim.x) a.zero[i] = 0;
}

// Byte-parallel comparison: bit 7 of byte b of the result is [u_b >= v_b]
// for unsigned bytes (the other bits are don't-care).  vlo = v & 0x7F7F7F7F.
// (u | 0x80) - (v & 0x7F) per byte lies in [1, 255], so no borrow crosses a
// byte, and its bit 7 compares the low 7 bits; the top bits decide whenever
// they differ.
__device__ inline uint32_t ge_bytes(uint32_t u, uint32_t v, uint32_t vlo) {
    const uint32_t d = (u | 0x80808080u) - vlo;
    return (u & ~v) | (~(u ^ v) & d);
}

// Moves each byte of acc down one bit and puts bit 7 of the byte of g on top.
__device__ inline uint32_t push_bits(uint32_t acc, uint32_t g) {
    return ((acc >> 1) & 0x7F7F7F7Fu) | (g & 0x80808080u);
}

// o[p] byte b = a[b] byte p (4x4 byte transpose).
__device__ inline void transpose_bytes4(const uint32_t (&a)[4], uint32_t (&o)[4]) {
    const uint32_t t01l = __builtin_amdgcn_perm(a[1], a[0], 0x05010400u);
    const uint32_t t01h = __builtin_amdgcn_perm(a[1], a[0], 0x07030602u);
    const uint32_t t23l = __builtin_amdgcn_perm(a[3], a[2], 0x05010400u);
    const uint32_t t23h = __builtin_amdgcn_perm(a[3], a[2], 0x07030602u);
    o[0] = __builtin_amdgcn_perm(t23l, t01l, 0x05040100u);
    o[1] = __builtin_amdgcn_perm(t23l, t01l, 0x07060302u);
    o[2] = __builtin_amdgcn_perm(t23h, t01h, 0x05040100u);
    o[3] = __builtin_amdgcn_perm(t23h, t01h, 0x07060302u);
}

// Census words (9x7 window, full or center-symmetric) of 4 consecutive
// pixels of one row, from a byte tile with row pitch TW (a multiple of 4).
// Pixel p (0..3) has its window on tile rows r0 .. r0+6 and columns
// c0+p .. c0+p+8 (centre at row r0+3, column c0+p+4); c0 is a multiple of 4,
// so each window row is read as 3 aligned dwords.
//
// The 4 pixels' samples at one window offset are 4 consecutive bytes of a
// tile row, so one dword holds them and ge_bytes compares all four.  Byte b
// of the census word (bits 8b .. 8b+7) is gathered for the 4 pixels in the
// 4 bytes of acc[b], one push_bits per bit; a byte transpose then turns the
// per-bit-byte registers into per-pixel words.
__device__ inline void census_words4(const uint8_t* tile, int TW, int r0, int c0, bool csct, uint64_t words[4]) {
    constexpr int RY = 3, CW = 9;
    uint32_t dw[2 * RY + 1][3];
#pragma unroll
    for (int j = 0; j < 2 * RY + 1; ++j)
#pragma unroll
        for (int k = 0; k < 3; ++k) dw[j][k] = *reinterpret_cast<const uint32_t*>(&tile[(r0 + j) * TW + c0 + 4 * k]);
    // bytes b .. b+3 of window row j (b in 0..8): column offset b - 4 of the 4 pixels
    auto at = [&](int j, int b) -> uint32_t {
        const int q = b >> 2, s = b & 3;
        return s == 0 ? dw[j][q] : __builtin_amdgcn_alignbit(dw[j][q + 1], dw[j][q], 8 * s);
    };
    uint32_t acc[8];
    if (!csct) {
        // bit k = (j, i) of the window: k = j * 9 + i, j in 0..6, i in 0..8
        const uint32_t c = at(RY, 4), clo = c & 0x7F7F7F7Fu;
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            uint32_t a = 0;
            const int nb = b < 7 ? 8 : (2 * RY + 1) * CW - 56;  // 7 bits in the top byte
#pragma unroll
            for (int t = 0; t < nb; ++t) {
                const int k = 8 * b + t;
                a = push_bits(a, ge_bytes(at(k / CW, k % CW), c, clo));
            }
            acc[b] = nb == 8 ? a : (a >> (8 - nb)) & (0xFFu >> (8 - nb)) * 0x01010101u;
        }
    } else {
        // pairs in order k = 0..30: i = 1..4 with j = -3..3, then (0, j), j = 1..3
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            uint32_t a = 0;
            const int nb = b < 3 ? 8 : 7;
#pragma unroll
            for (int t = 0; t < nb; ++t) {
                const int k = 8 * b + t;
                int i, j;
                if (k < 28) {
                    i = 1 + k / 7;
                    j = k % 7 - 3;
                } else {
                    i = 0;
                    j = k - 27;
                }
                const uint32_t u = at(RY + j, 4 + i), v = at(RY - j, 4 - i);
                a = push_bits(a, ge_bytes(u, v, v & 0x7F7F7F7Fu));
            }
            acc[b] = nb == 8 ? a : (a >> 1) & 0x7F7F7F7Fu;
        }
#pragma unroll
        for (int b = 4; b < 8; ++b) acc[b] = 0;
    }
    uint32_t lo[4], hi[4];
    transpose_bytes4({acc[0], acc[1], acc[2], acc[3]}, lo);
    transpose_bytes4({acc[4], acc[5], acc[6], acc[7]}, hi);
#pragma unroll
    for (int p = 0; p < 4; ++p) words[p] = ((uint64_t)hi[p] << 32) | lo[p];
}

__device__ inline void census97_block(const CensusArgs& a, int bx, int by, int z) {
    census_clear(a, bx, by, z);
    constexpr int RY = 3;
    constexpr int TW = kCenTX + 8, TH = kCenTY + 2 * RY;
    __shared__ __align__(16) uint8_t tile[TH * TW];

    const uint8_t* img = a.img[z];
    const int x0 = bx * kCenTX, y0 = by * kCenTY;
    // all loads first, then the LDS stores (the block has 256 threads)
    constexpr int kIt = (TH * TW + 255) / 256;
    uint32_t v[kIt];
#pragma unroll
    for (int k = 0; k < kIt; ++k) {
        const int i = threadIdx.x + 256 * k;
        const int r = i / TW, c = i - r * TW;
        const int yy = clampi(y0 - RY + r, 0, a.H - 1), xx = clampi(x0 - 4 + c, 0, a.W - 1);
        v[k] = i < TH * TW ? img[(size_t)yy * a.W + xx] : 0u;
    }
#pragma unroll
    for (int k = 0; k < kIt; ++k)
        if (threadIdx.x + 256 * k < TH * TW) tile[threadIdx.x + 256 * k] = (uint8_t)v[k];
    __syncthreads();
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    const int y = y0 + ty;
    uint64_t words[4];
    census_words4(tile, TW, ty, 4 * tx, a.csct != 0, words);
    const int x = x0 + 4 * tx;
    if (y < a.H) {
        uint64_t* o = a.out[z] + (size_t)y * a.W + x;
        if (x + 3 < a.W && ((a.W & 1) == 0)) {
            // plain (write-back) stores: a thread's two 16-byte stores fill
            // the two halves of its 32 bytes, which the L2 merges; with
            // device scope each half would be written through on its own
            reinterpret_cast<ulonglong2*>(o)[0] = make_ulonglong2(words[0], words[1]);
            reinterpret_cast<ulonglong2*>(o)[1] = make_ulonglong2(words[2], words[3]);
        } else {
#pragma unroll
            for (int p = 0; p < 4; ++p)
                if (x + p < a.W) o[p] = words[p];
        }
    }
}

// Any other window: one thread per pixel, straight from global memory.
__device__ inline void census_generic_block(const CensusArgs& a, int rx, int ry, int bx, int by, int z) {
    census_clear(a, bx, by, z);
    const int x = bx * 16 + (threadIdx.x & 15);
    const int y = by * 16 + (threadIdx.x >> 4);

    if (x >= a.W || y >= a.H) return;
    const uint8_t* img = a.img[z];
    auto at = [&](int i, int j) {
        return (int)img[(size_t)clampi(y + j, 0, a.H - 1) * a.W + clampi(x + i, 0, a.W - 1)];
    };
    const int cw = 2 * rx + 1;
    uint64_t word = 0;
    if (!a.csct) {
        const int c = at(0, 0);
        for (int j = -ry; j <= ry; ++j)
            for (int i = -rx; i <= rx; ++i)
                word |= (uint64_t)(at(i, j) >= c ? 1u : 0u) << ((j + ry) * cw + (i + rx));
    } else {
        int k = 0;
        for (int i = 1; i <= rx; ++i)
            for (int j = -ry; j <= ry; ++j, ++k) word |= (uint64_t)(at(i, j) >= at(-i, -j) ? 1u : 0u) << k;
        for (int j = 1; j <= ry; ++j, ++k) word |= (uint64_t)(at(0, j) >= at(0, -j) ? 1u : 0u) << k;
    }
    a.out[z][(size_t)y * a.W + x] = word;
}

// ---------------------------------------------------------------------------
// Matching cost (Eq. 2).  One wavefront per (row y, unit of PX base
// pixels).  A lane makes the costs of 16 consecutive disparities of one
// pixel after another, RUN pixels in all: 16 lanes (8, 4) hold the 256 (128, 64)
// levels of a pixel, and the wavefront works on pixels RUN apart.  From one pixel
// to the next a lane's 16 match words move on by one, so a step reads one match
// and one base word from LDS for 16 costs, and its 16 costs are one 16-byte
// store at the place they belong.  The unit's words are staged by the
// wavefront for itself: no barrier, and a block is four independent units.
//
// The VALU and the stores bound it about alike: two xor, two counting
// instructions and a shift per cost, against one byte.  1920x1080, D = 256: 88
// us (6.0 TB/s of costs; before, with a lane per pixel, a tile in LDS and a
// copy out of it, 113); 640x480, D = 128: 11.7 us (12.7); 64 mixed pairs,
// 2.6 GB: 711 us (967).
// ---------------------------------------------------------------------------
constexpr int kCostThreads = 256;  // block size of every launch of cost_unit
template <int DP, int RUN>
struct CostUnit {
    static constexpr int G = DP / 16;                  // lanes per pixel
    static constexpr int PX = 64 / G * RUN;            // pixels per unit
    static constexpr int N = 2 * PX + DP;              // words staged: PX base, PX + DP match
    static constexpr int words = N / RUN * (RUN + 1);  // in LDS: one word of padding after every RUN
};
__host__ __device__ constexpr int cost_unit_px(int Dp, int run) { return 64 / (Dp / 16) * run; }

struct CostArgs {
    const uint64_t* cl;
    const uint64_t* cr;
    uint8_t* cost;
    int W, H, D, Dp, cmax;
};

// RB = false: base words cl = left view, match words cr = right view at x - d
// (Eq. 2).  RB = true: base = right view, match = left view at x + d (the
// right-base costs of the full left-right check).  DP = a.Dp (64, 128 or 256).
// smem: CostUnit::words words of this wavefront's own.  AUX: store policy.
template <bool RB, int DP, int RUN, int AUX>
__device__ inline void cost_unit(const CostArgs& a, int ux, int y, int lane, uint64_t* smem) {
    using U = CostUnit<DP, RUN>;
    constexpr int G = U::G, PX = U::PX;
    const int x0 = ux * PX, W = a.W, D = a.D;
    // item n of the unit is base word x0 + n (n < PX) or match word
    // xm0 + n - PX, at LDS word n + n / RUN: the lanes of a step read words a
    // multiple of RUN apart, which the padding spreads over the banks
    const int xm0 = RB ? x0 : x0 - DP;
    const uint64_t* gl = a.cl + (size_t)y * W;
    const uint64_t* gr = a.cr + (size_t)y * W;
    constexpr int kLoads = (U::N + 63) / 64;
    uint64_t v[kLoads];
#pragma unroll
    for (int k = 0; k < kLoads; ++k) {
        const int n = lane + 64 * k;
        const bool base = n < PX;
        const int x = base ? x0 + n : xm0 + n - PX;
        v[k] = 0;
        if (x >= 0 && x < W && n < U::N) v[k] = (base ? gl : gr)[x];
    }
#pragma unroll
    for (int k = 0; k < kLoads; ++k) {
        const int n = lane + 64 * k;
        if (n < U::N) smem[n + n / RUN] = v[k];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();

    const int g = lane / G, q = lane % G;
    constexpr int PR = RUN + 1, HOP = 16 / RUN;
    const uint64_t* bl = smem + PR * g;
    // match word of step s, disparity 16q + j: column x - 16q - j, item
    // PX + DP + RUN g - 16q + (s - j) (left base), or x + 16q + j, item
    // PX + RUN g + 16q + (s + j)
    const uint64_t* ml = smem + PR * (PX / RUN + (RB ? g + HOP * q : DP / RUN + g - HOP * q));
    auto word = [&](int o) { return ml[PR * ((o + 16) / RUN - HOP) + (o + 16) % RUN]; };  // o >= -15
    const int col = x0 + RUN * g + (RB ? 16 * q : -16 * q);  // match column of s = j = 0
    uint8_t* const row = a.cost + (size_t)y * W * DP;
    const uint32_t ofs = (uint32_t)((x0 + RUN * g) * DP + 16 * q);  // past the row's end: dropped

    auto run = [&](auto general) {
        constexpr bool GENERAL = decltype(general)::value;
        // Levels d >= D get kPadCost and match pixels outside the image Cmax.
        // Both are byte masks over the 16 levels; the second moves on by a
        // byte a step (the last levels of a lane are outside, fewer of them
        // with every step to the right and more with the right base), so it
        // extends past the 16 by the bytes that move in.
        constexpr int E = (RUN + 3) / 4;
        // 0xFF in the bytes of word k from byte n on (bytes counted from word 0)
        auto from = [](int n, int k) { return (uint32_t)(~0ull << (8 * min(max(n - 4 * k, 0), 4))); };
        uint32_t pad[4], out[4 + E];  // out[k]: word k - E (left base) or k of the mask
        if constexpr (GENERAL) {
#pragma unroll
            for (int k = 0; k < 4; ++k) pad[k] = from(D - 16 * q, k);
#pragma unroll
            for (int k = 0; k < 4 + E; ++k) out[k] = RB ? from(W - col, k) : from(col + 1, k - E);
        }
        uint64_t w[16];  // the window: word o in slot o & 15
#pragma unroll
        for (int j = 0; j < 16; ++j) w[(RB ? j : -j) & 15] = word(RB ? j : -j);
#pragma unroll
        for (int s = 0; s < RUN; ++s) {
            const uint64_t b = bl[s];
            uint32_t c[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                c[k] = 0;
#pragma unroll
                for (int i = 3; i >= 0; --i) {
                    const int j = 4 * k + i;
                    const uint64_t x = b ^ w[(RB ? s + j : s - j) & 15];
                    c[k] = (uint32_t)__popc((uint32_t)(x >> 32)) + ((uint32_t)__popc((uint32_t)x) + (c[k] << 8));
                }
                if constexpr (GENERAL) {
                    const uint32_t o = out[RB ? k : k + E];
                    c[k] = ((uint32_t)a.cmax * 0x01010101u & o) | (c[k] & ~o);
                    c[k] = (kPadCost * 0x01010101u & pad[k]) | (c[k] & ~pad[k]);
                }
            }
            if (s + 1 < RUN) {
                const int o = RB ? s + 16 : s + 1;
                w[o & 15] = word(o);
                if constexpr (GENERAL) {
                    if constexpr (RB) {
#pragma unroll
                        for (int k = 0; k < 4 + E; ++k)
                            out[k] = __builtin_amdgcn_alignbit(k + 1 < 4 + E ? out[k + 1] : ~0u, out[k], 8);
                    } else {
#pragma unroll
                        for (int k = 3 + E; k >= 0; --k)
                            out[k] = __builtin_amdgcn_alignbit(out[k], k > 0 ? out[k - 1] : 0u, 24);
                    }
                }
            }
            store16<AUX>(row, (uint32_t)(W * DP), ofs + (uint32_t)(s * DP), make_uint4(c[0], c[1], c[2], c[3]));
        }
    };
    const bool border = RB ? x0 + PX - 1 + D - 1 >= W : x0 < D - 1;
    if (border || D < DP)
        run(std::true_type{});
    else
        run(std::false_type{});
}

// ---------------------------------------------------------------------------
// Census + matching cost in one pass (9x7 windows).  One block per (row y,
// segment of kCcRuns runs of 64 base pixels).  The block stages the 7 image
// rows around y of both views in LDS (clamp-to-edge): the base view over the
// segment, the match view over the segment plus the D - 1 columns to its
// left.  It computes every census word it needs exactly once into LDS, then
// for each run of 64 pixels builds the costs in an LDS tile [64][Dp + 16]
// (two tiles, alternating, so one run's copy-out overlaps the next run's
// popcounts) and writes the run's slice of the cost volume with contiguous
// 16-byte stores.  No census word goes through global memory.
// ---------------------------------------------------------------------------
constexpr int kCcRuns = 4;
constexpr int kCcTX = 64 * kCcRuns;

struct CensusCostArgs {
    const uint8_t* left;
    const uint8_t* right;
    uint8_t* cost;
    int W, H, D, Dp, cmax, csct;
    int* zero = nullptr;  // as CensusArgs::zero
    int nzero = 0;
};

// Byte sizes of the LDS regions of census_cost_block.
struct CcLayout {
    int twl, twr;     // tile row pitches (bytes), base / match view
    int nr;           // match census words: kCcTX + D - 1, rounded up to 4
    int words_off;    // byte offset of the census words (base, then match)
    int tiles_off;    // byte offset of the two cost tiles
    int tpitch;       // bytes per cost-tile row
    int bytes;        // total
};

__host__ __device__ inline CcLayout cc_layout(int D, int Dp) {
    CcLayout L;
    L.twl = kCcTX + 8;
    L.nr = (kCcTX + D - 1 + 3) & ~3;
    L.twr = L.nr + 8;
    L.words_off = (7 * (L.twl + L.twr) + 15) & ~15;
    L.tiles_off = L.words_off + 8 * (kCcTX + L.nr);
    L.tpitch = Dp + 16;
    L.bytes = L.tiles_off + 2 * 64 * L.tpitch;
    return L;
}

__device__ inline void census_cost_block(const CensusCostArgs& a, int bx, int y, uint8_t* smem) {
    if (a.zero && (bx | y) == 0)
        for (int i = threadIdx.x; i < a.nzero; i += blockDim.x) a.zero[i] = 0;
    constexpr int RY = 3;
    const int D = a.D, Dp = a.Dp;
    const CcLayout L = cc_layout(D, Dp);
    const int x0 = bx * kCcTX;
    const int xs = x0 - (D - 1);  // first match column
    uint8_t* tl = smem;           // base view tile: 7 rows, columns x0 - 4 ..
    uint8_t* tr = smem + 7 * L.twl;  // match view tile: 7 rows, columns xs - 4 ..
    uint64_t* cl = reinterpret_cast<uint64_t*>(smem + L.words_off);  // cl[i]: column x0 + i
    uint64_t* cr = cl + kCcTX;                                        // cr[i]: column xs + i
    uint8_t* tiles = smem + L.tiles_off;

    // Stage the 7 image rows of both views.  Every load is issued before the
    // first LDS store, so the loads' latencies overlap instead of adding up
    // (the block has 256 threads; a base row has kCcTX + 8 <= 512 bytes, a
    // match row at most 520 <= 768).
    {
        const int t = threadIdx.x;
        uint32_t vl[7][2], vr[7][3];
#pragma unroll
        for (int r = 0; r < 7; ++r) {
            const size_t row = (size_t)clampi(y - RY + r, 0, a.H - 1) * a.W;
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int c = t + 256 * k;
                vl[r][k] = c < L.twl ? a.left[row + clampi(x0 - 4 + c, 0, a.W - 1)] : 0u;
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const int c = t + 256 * k;
                vr[r][k] = c < L.twr ? a.right[row + clampi(xs - 4 + c, 0, a.W - 1)] : 0u;
            }
        }
#pragma unroll
        for (int r = 0; r < 7; ++r) {
#pragma unroll
            for (int k = 0; k < 2; ++k)
                if (t + 256 * k < L.twl) tl[r * L.twl + t + 256 * k] = (uint8_t)vl[r][k];
#pragma unroll
            for (int k = 0; k < 3; ++k)
                if (t + 256 * k < L.twr) tr[r * L.twr + t + 256 * k] = (uint8_t)vr[r][k];
        }
    }
    __syncthreads();
    {
        const int nl4 = kCcTX / 4, nr4 = L.nr / 4;
        for (int t = threadIdx.x; t < nl4 + nr4; t += blockDim.x) {
            uint64_t w[4];
            if (t < nl4) {
                census_words4(tl, L.twl, 0, 4 * t, a.csct != 0, w);
#pragma unroll
                for (int p = 0; p < 4; ++p) cl[4 * t + p] = w[p];
            } else {
                const int u = t - nl4;
                census_words4(tr, L.twr, 0, 4 * u, a.csct != 0, w);
#pragma unroll
                for (int p = 0; p < 4; ++p) cr[4 * u + p] = w[p];
            }
        }
    }
    __syncthreads();

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwaves = blockDim.x >> 6;
    const int nchunks = Dp >> 4;
    for (int run = 0; run < kCcRuns; ++run) {
        const int xr0 = x0 + 64 * run;
        if (xr0 >= a.W) break;  // the same for the whole block
        uint8_t* tile = tiles + (run & 1) * 64 * L.tpitch;
        const int x = xr0 + lane;
        const uint64_t base = cl[64 * run + lane];
        for (int ch = wave; ch < nchunks; ch += nwaves) {
            const int d0 = 16 * ch;
            // match word of disparity d0 + j is cr[64 run + lane + D - 1 - d0 - j]
            const uint64_t* m = cr + (64 * run + lane + D - 1 - d0 - 15);
            uint32_t w[4];
            if (xr0 >= d0 + 15 && d0 + 16 <= D) {  // all 16 disparities valid for every lane
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    uint32_t word = 0;
#pragma unroll
                    for (int j = 0; j < 4; ++j) word |= (uint32_t)__popcll(base ^ m[15 - (4 * q + j)]) << (8 * j);
                    w[q] = word;
                }
            } else if (d0 + 16 <= D) {  // at the border: popcount on every lane, then a select
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    uint32_t word = 0;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const uint32_t pc = (uint32_t)__popcll(base ^ m[15 - (4 * q + j)]);
                        word |= (x - (d0 + 4 * q + j) < 0 ? (uint32_t)a.cmax : pc) << (8 * j);
                    }
                    w[q] = word;
                }
            } else {  // the chunk holding D - 1 and the padded levels
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    uint32_t word = 0;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int d = d0 + 4 * q + j;
                        uint32_t c = kPadCost;  // padded levels d >= D
                        if (d < D) {
                            const uint32_t pc = (uint32_t)__popcll(base ^ m[15 - (4 * q + j)]);
                            c = x - d < 0 ? (uint32_t)a.cmax : pc;
                        }
                        word |= c << (8 * j);
                    }
                    w[q] = word;
                }
            }
            *reinterpret_cast<uint4*>(tile + lane * L.tpitch + d0) = make_uint4(w[0], w[1], w[2], w[3]);
        }
        __syncthreads();
        const int npx = min(64, a.W - xr0);
        const int lg = Dp == 64 ? 2 : (Dp == 128 ? 3 : 4);  // log2(nchunks)
        uint8_t* dst = a.cost + ((size_t)y * a.W + xr0) * Dp;
        for (int c = threadIdx.x; c < npx * nchunks; c += blockDim.x) {
            const int px = c >> lg, k = c & (nchunks - 1);
            store16(dst, (uint32_t)(npx * Dp), 16u * (uint32_t)c,
                        *reinterpret_cast<const uint4*>(tile + px * L.tpitch + 16 * k));
        }
    }
}

// ---------------------------------------------------------------------------
// Aggregation (Eq. 3).
//
// The recurrence forbids parallelism along a path (Sec. 3.2), so the work is
// spread over slices x disparities x directions.  A group of G lanes (G in
// {16, 32, 64}) owns one slice and walks it step by step; a wavefront holds
// S = 64 / G slices of the same direction.  Lane q of a group holds the
// disparities q*CPL .. q*CPL + CPL - 1 (CPL = Dp / G) of L_r(p - r, .) as
// CPL/2 packed u16 pairs in a "split" layout: pair k holds disparities
// q*CPL + k (low half) and q*CPL + k + CPL/2 (high half), so the d-1 / d+1
// neighbours of pair k are pairs k-1 / k+1 of the same lane, except at the
// lane's two ends, which take one DPP lane shift and one v_alignbit each.
// Per step, with m = min_k L(p - r, k) and R(d) = min(L(p - r, d),
// L(p - r, d +- 1) + P1) left by the step before:
//   L'(d) = C(p, d) + min(R(d) - m, P2)     (Eq. 3; R >= m)
//   R'(d) = min(L'(d), L'(d +- 1) + P1)
//   m'    = min_d L'(d)                     (group min-reduction)
// so the chain from m to m' is subtract, minimum, add and the reduction, and
// R' is formed beside the reduction.  "No such disparity" (the d-1 of d = 0,
// the d+1 of d = D-1, padded levels d >= D) is 0xFFFF in saturating u16
// arithmetic on 16-bit planes, and a finite stand-in on byte planes (below).
// Real values are at most Cmax + 2*P2 < 0xFFFF (validated), so saturation
// never changes a result.  A path start is R = 0 and m = 0, which makes
// L' = C exactly.
//
// What bounds it: frames whose slices give each SIMD one wavefront or less
// are bound by a step's length (72 ns for a 32-lane horizontal step, 31
// instructions; 95 ns for a 16-lane vertical one, 44), the others by the
// bytes.  Against the schedule the compiler chose by itself (86 and 114 ns):
// 4 directions of 640x480, D = 128, alone on the device 56.1 -> 47.7 us
// (5.6 -> 6.6 TB/s), its 4 diagonals 86.7 -> 53.7 us, 320x240, D = 64
// 30.1 -> 22.3 us, 8 directions of 1242x375, D = 128 179.7 -> 164.2 us.
// ---------------------------------------------------------------------------
// Everything one wavefront needs to aggregate slices of one direction.
struct SliceArgs {
    const uint8_t* cost;       // C u8 [H][W][Dp] (cost-volume variant)
    const uint64_t* census_l;  // census words (fused variant)
    const uint64_t* census_r;
    void* lplane;              // this direction's L_r plane [H][W][Dp]
    uint32_t plane;            // elements per plane = H * W * Dp
    int W, H, D, P1, P2, cmax, rx, ry;
    const uint8_t* img = nullptr;      // base image u8 [H][W] (adaptive P2)
    const uint16_t* p2lut = nullptr;   // LDS: adaptive P2 of each intensity change 0..255
};

// Adaptive P2 of one step: max(P1, floor(P2 / (1 + g))) for an intensity
// change g in [0, 255].  A block tabulates it once in LDS (fill_p2_lut) and
// the recurrence looks values up.
__device__ inline uint32_t adaptive_p2(uint32_t P1, uint32_t P2, uint32_t g) {
    const uint32_t q = P2 / (1u + g);
    return q > P1 ? q : P1;
}

// Fills lut[0..255] with adaptive_p2 (all threads of the block take part;
// the caller synchronizes before use).
__device__ inline void fill_p2_lut(uint16_t* lut, int P1, int P2) {
    for (int g = threadIdx.x; g < 256; g += blockDim.x) lut[g] = (uint16_t)adaptive_p2((uint32_t)P1, (uint32_t)P2, (uint32_t)g);
}

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
__device__ inline u16x2 as2(uint32_t v) { return __builtin_bit_cast(u16x2, v); }
__device__ inline uint32_t as1(u16x2 v) { return __builtin_bit_cast(uint32_t, v); }
__device__ inline u16x2 vmin(u16x2 a, u16x2 b) { return __builtin_elementwise_min(a, b); }
__device__ inline u16x2 vadds(u16x2 a, u16x2 b) { return __builtin_elementwise_add_sat(a, b); }

// Minimum of three packed u16 pairs in one v_pk_minimum3_f16.  Exact for
// halves below 0x7C00: those bit patterns are the non-negative finite f16
// values (zero, subnormals, normals), whose order is the order of the
// patterns read as unsigned integers, and a minimum returns one of its
// inputs unchanged.  f16 subnormals are not flushed in these kernels (the
// f16/f64 denormal mode keeps them), so small integers compare correctly.
typedef _Float16 h16x2 __attribute__((ext_vector_type(2)));
__device__ inline u16x2 vmin3h(u16x2 a, u16x2 b, u16x2 c) {
    const h16x2 m = __builtin_elementwise_minimum(__builtin_elementwise_minimum(__builtin_bit_cast(h16x2, a),
                                                                                __builtin_bit_cast(h16x2, b)),
                                                  __builtin_bit_cast(h16x2, c));
    return __builtin_bit_cast(u16x2, m);
}

// DPP controls (GFX9 encoding).
constexpr int kDppQuadPerm1032 = 0xB1;
constexpr int kDppQuadPerm2301 = 0x4E;
constexpr int kDppRowShl1 = 0x101;   // lane i reads lane i+1 within a row of 16
constexpr int kDppRowShr1 = 0x111;   // lane i reads lane i-1 within a row of 16
constexpr int kDppWaveShl1 = 0x130;  // lane i reads lane i+1
constexpr int kDppWaveShr1 = 0x138;  // lane i reads lane i-1
constexpr int kDppRowMirror = 0x140;
constexpr int kDppRowHalfMirror = 0x141;

// Lane j's value of each row of 16 lanes, in all lanes of the row
// (row_newbcast; j is a constant once the caller's loop is unrolled).
__device__ __attribute__((always_inline)) inline uint32_t row_broadcast(uint32_t v, int j) {
#define SGM_ROW_BCAST(J) \
    case J: return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x150 + J, 0xF, 0xF, true);
    switch (j & 15) {
        SGM_ROW_BCAST(0) SGM_ROW_BCAST(1) SGM_ROW_BCAST(2) SGM_ROW_BCAST(3) SGM_ROW_BCAST(4) SGM_ROW_BCAST(5)
        SGM_ROW_BCAST(6) SGM_ROW_BCAST(7) SGM_ROW_BCAST(8) SGM_ROW_BCAST(9) SGM_ROW_BCAST(10) SGM_ROW_BCAST(11)
        SGM_ROW_BCAST(12) SGM_ROW_BCAST(13) SGM_ROW_BCAST(14) default: break;
    }
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x15F, 0xF, 0xF, true);
#undef SGM_ROW_BCAST
}

// Lane q of a group receives lane q-1's (from_lower) or q+1's (from_upper)
// value; a lane without a source receives 0 (bound_ctrl), and group edges are
// overwritten by the caller's OR mask.
template <int G>
__device__ inline uint32_t from_lower(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, G == 16 ? kDppRowShr1 : kDppWaveShr1, 0xF, 0xF, true);
}
template <int G>
__device__ inline uint32_t from_upper(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, G == 16 ? kDppRowShl1 : kDppWaveShl1, 0xF, 0xF, true);
}

// Minimum over each group of G lanes; every lane of the group receives it.
// The butterfly inside a row of 16 uses DPP (folded into v_min_u32_dpp);
// groups spanning 2 or 4 rows combine rows with the gfx950 permlane swaps.
// fill<i>() runs between stages i - 1 and i (0 .. 3): independent work for
// the two wait states a DPP operand needs after it is written.
struct NoFill {
    template <int I> __device__ void operator()(std::integral_constant<int, I>) const {}
};
template <int G, typename FILL = NoFill>
__device__ inline uint32_t group_min(uint32_t v, FILL fill = FILL{}) {
    fill(std::integral_constant<int, 0>{});
    v = min(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kDppQuadPerm1032, 0xF, 0xF, true));
    fill(std::integral_constant<int, 1>{});
    v = min(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kDppQuadPerm2301, 0xF, 0xF, true));
    fill(std::integral_constant<int, 2>{});
    v = min(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kDppRowHalfMirror, 0xF, 0xF, true));
    fill(std::integral_constant<int, 3>{});
    v = min(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kDppRowMirror, 0xF, 0xF, true));
    if constexpr (G >= 32) {
        const auto sw = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        v = min((uint32_t)sw[0], (uint32_t)sw[1]);
    }
    if constexpr (G == 64) {
        const auto sw = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        v = min((uint32_t)sw[0], (uint32_t)sw[1]);
    }
    return v;
}

// The same reduction with a bitwise or (G = 16 or 32).
template <int G>
__device__ inline uint32_t group_or(uint32_t v) {
    v |= (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kDppQuadPerm1032, 0xF, 0xF, true);
    v |= (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kDppQuadPerm2301, 0xF, 0xF, true);
    v |= (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kDppRowHalfMirror, 0xF, 0xF, true);
    v |= (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kDppRowMirror, 0xF, 0xF, true);
    if constexpr (G == 32) {
        const auto sw = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        v = (uint32_t)sw[0] | (uint32_t)sw[1];
    }
    return v;
}

// Raw cost bytes of one lane for one step: CPL bytes.
template <int CPL> struct Raw;
template <> struct Raw<2> { using T = uint16_t; };
template <> struct Raw<4> { using T = uint32_t; };
template <> struct Raw<8> { using T = uint2; };
template <> struct Raw<16> { using T = uint4; };

// Unpacks a lane's cost bytes b_0..b_{CPL-1} into pairs (b_k, b_{k+CPL/2})
// with one v_perm per pair.  sel[k] is the per-lane byte selector; it selects
// 0xFF bytes for padded levels, which makes their cost 0xFFFF.
template <int CPL>
__device__ inline void unpack_costs(const typename Raw<CPL>::T& r, const uint32_t (&sel)[CPL / 2],
                                    u16x2 (&c)[CPL / 2]) {
    if constexpr (CPL == 2) {
        c[0] = as2(__builtin_amdgcn_perm(0u, (uint32_t)r, sel[0]));
    } else if constexpr (CPL == 4) {
        c[0] = as2(__builtin_amdgcn_perm(r, r, sel[0]));
        c[1] = as2(__builtin_amdgcn_perm(r, r, sel[1]));
    } else if constexpr (CPL == 8) {
#pragma unroll
        for (int k = 0; k < 4; ++k) c[k] = as2(__builtin_amdgcn_perm(r.y, r.x, sel[k]));
    } else {
        const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
        for (int k = 0; k < 8; ++k) c[k] = as2(__builtin_amdgcn_perm(w[2 + k / 4], w[k / 4], sel[k]));
    }
}

// Selector of pair k for a lane whose first disparity is d0: low half b_k,
// high half b_{k+CPL/2} (bytes of the v_perm source pair); for d >= D
// 0x03FF (the level's own byte kPadCost above 0xFF) with `byte_planes`, else
// 0xFFFF.
template <int CPL>
__device__ inline uint32_t unpack_selector(int k, int d0, int D, bool byte_planes) {
    constexpr int NP = CPL / 2;
    uint32_t lo, hi;
    if constexpr (CPL == 2) {
        lo = 0;
        hi = 1;
    } else if constexpr (CPL == 4) {
        lo = k;
        hi = k + 2;
    } else {
        lo = k % 4;
        hi = 4 + k % 4;
    }
    const uint32_t slo = (d0 + k < D) ? (lo | 0x0C00u) : (byte_planes ? (lo << 8) | 0x0Du : 0x0D0Du);
    const uint32_t shi = (d0 + k + NP < D) ? (hi | 0x0C00u) : (byte_planes ? (hi << 8) | 0x0Du : 0x0D0Du);
    return slo | (shi << 16);
}

enum { kHoriz = 0, kVert = 1, kDiag = 2 };

// Raw-buffer resource for a byte range (gfx9-family descriptor word 3).
// Accesses that rely on the hardware range check (loads past `bytes` return 0
// and stores past it are dropped) pass their whole byte offset in the VGPR
// operand; the aggregation's loads and stores stay inside the buffers by
// themselves and put the part of the offset that is the same for the whole
// wavefront into the scalar operand.
__device__ inline __amdgpu_buffer_rsrc_t buffer_rsrc(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}

template <int CPL>
__device__ inline typename Raw<CPL>::T buffer_load_raw(__amdgpu_buffer_rsrc_t r, uint32_t ofs, uint32_t sofs) {
    if constexpr (CPL == 2) {
        return (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r, ofs, sofs, 0);
    } else if constexpr (CPL == 4) {
        return __builtin_amdgcn_raw_buffer_load_b32(r, ofs, sofs, 0);
    } else if constexpr (CPL == 8) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, ofs, sofs, 0);
        return make_uint2(v[0], v[1]);
    } else {
        const auto v = __builtin_amdgcn_raw_buffer_load_b128(r, ofs, sofs, 0);
        return make_uint4(v[0], v[1], v[2], v[3]);
    }
}

// AUX is the cache-policy operand of the store (gfx950: 2 = non-temporal,
// 16 = device scope, sc1).
template <int AUX>
__device__ inline void buffer_store(__amdgpu_buffer_rsrc_t r, uint32_t ofs, uint32_t sofs, uint16_t v) {
    __builtin_amdgcn_raw_buffer_store_b16(v, r, ofs, sofs, AUX);
}
template <int AUX>
__device__ inline void buffer_store(__amdgpu_buffer_rsrc_t r, uint32_t ofs, uint32_t sofs, uint32_t v) {
    __builtin_amdgcn_raw_buffer_store_b32(v, r, ofs, sofs, AUX);
}
template <int AUX>
__device__ inline void buffer_store(__amdgpu_buffer_rsrc_t r, uint32_t ofs, uint32_t sofs, uint2 v) {
    __builtin_amdgcn_raw_buffer_store_b64((unsigned __attribute__((ext_vector_type(2)))){v.x, v.y}, r, ofs, sofs, AUX);
}
template <int AUX>
__device__ inline void buffer_store(__amdgpu_buffer_rsrc_t r, uint32_t ofs, uint32_t sofs, uint4 v) {
    __builtin_amdgcn_raw_buffer_store_b128((unsigned __attribute__((ext_vector_type(4)))){v.x, v.y, v.z, v.w}, r, ofs,
                                           sofs, AUX);
}

// A lane's CPL L values as bytes in natural disparity order (u8 planes):
// pair k holds disparities k and k + CPL/2 (split layout), so the bytes are
// gathered with v_perm.
template <int CPL>
__device__ inline typename Raw<CPL>::T pack_u8(const u16x2 (&l)[CPL / 2]) {
    constexpr uint32_t kLoBytes = 0x06020400u;  // (a.b0, b.b0, a.b2, b.b2) of perm(b, a)
    constexpr uint32_t kPairLo = 0x05040100u;   // (a.lo16, b.lo16)
    constexpr uint32_t kPairHi = 0x07060302u;   // (a.hi16, b.hi16)
    if constexpr (CPL == 2) {
        return (uint16_t)__builtin_amdgcn_perm(0u, as1(l[0]), 0x0C0C0200u);
    } else if constexpr (CPL == 4) {
        return (uint32_t)__builtin_amdgcn_perm(as1(l[1]), as1(l[0]), kLoBytes);
    } else if constexpr (CPL == 8) {
        const uint32_t t01 = __builtin_amdgcn_perm(as1(l[1]), as1(l[0]), kLoBytes);
        const uint32_t t23 = __builtin_amdgcn_perm(as1(l[3]), as1(l[2]), kLoBytes);
        return make_uint2(__builtin_amdgcn_perm(t23, t01, kPairLo), __builtin_amdgcn_perm(t23, t01, kPairHi));
    } else {
        uint32_t t[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) t[i] = __builtin_amdgcn_perm(as1(l[2 * i + 1]), as1(l[2 * i]), kLoBytes);
        return make_uint4(__builtin_amdgcn_perm(t[1], t[0], kPairLo), __builtin_amdgcn_perm(t[3], t[2], kPairLo),
                          __builtin_amdgcn_perm(t[1], t[0], kPairHi), __builtin_amdgcn_perm(t[3], t[2], kPairHi));
    }
}

// Packs a lane's L values in natural disparity order (u8 or u16) and stores
// them at byte offset `ofs` (per lane) + `sofs` of the L_r plane.  NT: non-temporal stores (the
// frame's planes exceed the memory-side cache); otherwise device-scope (sc1)
// stores, which measured faster than plain ones: the planes still reach the
// memory-side cache for the WTA, and the L2 keeps more of the cost lines
// that the opposite direction of a slice re-reads.
template <int CPL, typename LT, bool NT = false>
__device__ inline void store_l(__amdgpu_buffer_rsrc_t r, uint32_t ofs, uint32_t sofs, const u16x2 (&l)[CPL / 2]) {
    constexpr int A = NT ? 2 : 16;
    constexpr uint32_t kPairLo = 0x05040100u;   // (a.lo16, b.lo16)
    constexpr uint32_t kPairHi = 0x07060302u;   // (a.hi16, b.hi16)
    if constexpr (sizeof(LT) == 1) {
        buffer_store<A>(r, ofs, sofs, pack_u8<CPL>(l));
    } else {
        constexpr int NP = CPL / 2;
        if constexpr (CPL == 2) {
            buffer_store<A>(r, ofs, sofs, as1(l[0]));
        } else {
            // dword i = (d_2i, d_2i+1) from pairs 2i and 2i+1 (low halves,
            // then high halves)
            uint32_t w[NP];
#pragma unroll
            for (int i = 0; i < NP / 2; ++i) {
                w[i] = __builtin_amdgcn_perm(as1(l[2 * i + 1]), as1(l[2 * i]), kPairLo);
                w[NP / 2 + i] = __builtin_amdgcn_perm(as1(l[2 * i + 1]), as1(l[2 * i]), kPairHi);
            }
            if constexpr (NP == 2) {
                buffer_store<A>(r, ofs, sofs, make_uint2(w[0], w[1]));
            } else {
#pragma unroll
                for (int i = 0; i < NP / 4; ++i)
                    buffer_store<A>(r, ofs + 16 * i, sofs, make_uint4(w[4 * i], w[4 * i + 1], w[4 * i + 2], w[4 * i + 3]));
            }
        }
    }
}

// Census words one lane needs for one step of the fused variant: the base
// word of its group's pixel and the CPL match words of columns x - d for its
// disparities d = q*CPL .. q*CPL + CPL - 1 (contiguous, lowest column first).
template <int CPL>
struct CensusStep {
    uint64_t base;
    uint64_t m[CPL];
};

template <int CPL>
__device__ inline void load_census(__amdgpu_buffer_rsrc_t rcl, __amdgpu_buffer_rsrc_t rcr, uint32_t base_ofs,
                                   uint32_t match_ofs, CensusStep<CPL>& cs) {
    const auto b = __builtin_amdgcn_raw_buffer_load_b64(rcl, base_ofs, 0, 0);
    cs.base = ((uint64_t)b[1] << 32) | b[0];
#pragma unroll
    for (int i = 0; i < CPL / 2; ++i) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b128(rcr, match_ofs + 16 * i, 0, 0);
        cs.m[2 * i] = ((uint64_t)v[1] << 32) | v[0];
        cs.m[2 * i + 1] = ((uint64_t)v[3] << 32) | v[2];
    }
}

// Hamming costs (Eq. 2) of a lane's CPL disparities, packed as the u16 pairs
// of the split layout.  Cell c (disparity q*CPL + c) uses match word
// m[CPL - 1 - c]; cells with c > valid_c (x - d < 0) cost cmax.  sel[k] puts
// the costs of cells k and k + CPL/2 into the two halves of pair k, or 0xFFFF
// for padded levels.
template <int CPL, bool ALL_VALID>
__device__ inline void census_costs(const CensusStep<CPL>& cs, int valid_c, uint32_t cmax,
                                    const uint32_t (&sel)[CPL / 2], u16x2 (&c)[CPL / 2]) {
    constexpr int NP = CPL / 2;
    uint32_t pc[CPL];
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
        const uint64_t x = cs.base ^ cs.m[CPL - 1 - i];
        pc[i] = (uint32_t)__popcll(x);
        if constexpr (!ALL_VALID) pc[i] = i > valid_c ? cmax : pc[i];
    }
#pragma unroll
    for (int k = 0; k < NP; ++k) c[k] = as2(__builtin_amdgcn_perm(pc[k + NP], pc[k], sel[k]));
}

// Selector of pair k for the fused variant: low half = cell k (S1 byte 0),
// high half = cell k + CPL/2 (S0 byte 0, selector 4); `pad` for d >= D.
template <int CPL>
__device__ inline uint32_t pack_selector(int k, int d0, int D, uint32_t pad) {
    constexpr int NP = CPL / 2;
    const uint32_t slo = (d0 + k < D) ? 0x0C00u : pad;
    const uint32_t shi = (d0 + k + NP < D) ? 0x0C04u : pad;
    return slo | (shi << 16);
}

// Cost loads run PF steps ahead of the recurrence so that their latency
// overlaps the dependent min-plus chain of the steps in between.
template <int CPL> struct Prefetch { static constexpr int N = CPL >= 16 ? 8 : 16; };
template <int CPL> struct FusedPrefetch { static constexpr int N = CPL >= 16 ? 2 : 4; };

// Where aggregate_wave puts each step's values E = L - C in [0, P2]: by
// default the direction's plane in global memory; with CkptSink only every
// kRowSegment-th column of it (horizontal directions: the states the row
// kernel starts from).  A sink (the final pass's LDS ring) instead receives
// put(step, E) for every step and chunk_done() after every Prefetch steps and
// after the last step.  (The census-computing variant stores L.)
struct PlaneSink {};
struct CkptSink {};

// Columns per segment of the row kernel, which runs both horizontal
// directions again inside every segment: a horizontal direction keeps its
// values only where it enters a segment.
template <int Dp, typename LT>
struct RowSegment {
    static constexpr int N = sizeof(LT) == 2 ? 8 : 16;
};

// A slice in segments: S wavefronts of one workgroup (S = 1: the whole slice).
//
// Segment 0 starts the path; the others start in the middle from an arbitrary
// state (a path start), so what they store is provisional.  Once every
// wavefront of the workgroup has walked its segment, each goes on into the
// next one, from its own end state, and overwrites what is stored there until
// it meets an equal value vector: equal E at one pixel is equal L there (the
// costs are the same), and from equal L the recurrence gives equal values, so
// the rest of that segment stands.  A wavefront that reaches a segment's end
// without meeting one goes on into the segment after it in the next round,
// when the other wavefronts' walks there have ended; segment 0's wavefront
// carries the true values, so after at most S - 1 rounds every segment holds
// them, whatever the costs.  On matched images the values meet within 10 to 50
// steps (a path that follows the surface forgets its start as soon as the
// other levels lie P2 above it); on unrelated images they may not meet at all
// and the slice takes its full length again.
//
// The point is the chain: a slice's dependent steps are divided by almost S.
struct Split {
    int seg = 0, S = 1;
    int* open = nullptr;  // LDS, one int per wavefront of the workgroup
    int wave = 0;         // of the workgroup's 4

    // One round's end for a wavefront that goes on (all wavefronts of the
    // workgroup take part in every round).  Its stores have completed before
    // the others read them.
    __device__ void next_round() const {
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
        open[wave] = 1;
        __syncthreads();
        __syncthreads();
    }
    // Rounds of a wavefront that has ended, until all have.
    __device__ void finish() const {
        if (S == 1) return;
        __builtin_amdgcn_s_waitcnt(0x0F70);
        for (;;) {
            open[wave] = 0;
            __syncthreads();
            const int any = open[0] | open[1] | open[2] | open[3];
            __syncthreads();
            if (__builtin_amdgcn_readfirstlane(any) == 0) return;
        }
    }
};

// ADAPT: the P2 of each step adapts to the base image's intensity change
// along the path (adaptive_p2): a block's intensities are loaded a block ahead,
// one step per lane, and looked up once per block.
template <int G, int CPL, typename LT, int KIND, bool FUSED, bool ADAPT = false, bool NT = false,
          typename SINK = PlaneSink, bool SPLIT = false>
__device__ inline void aggregate_wave(const SliceArgs& a, int first_slice, int lane, SINK* sink = nullptr,
                                      const Split& split = Split{}) {
    constexpr bool kCkpt = std::is_same_v<SINK, CkptSink>;
    constexpr bool kToPlane = std::is_same_v<SINK, PlaneSink> || kCkpt;
    static_assert(!kCkpt || (KIND == kHoriz && !FUSED), "checkpoints are for horizontal directions");
    static_assert(!SPLIT || (kToPlane && !FUSED && sizeof(LT) == 1 && KIND != kDiag),
                  "segments are for byte planes of L - C of axis-aligned directions");
    static_assert(!(FUSED && ADAPT), "adaptive P2 uses the cost-volume variant");
    constexpr int NP = CPL / 2;
    constexpr int Dp = G * CPL;
    constexpr int PF = FUSED ? FusedPrefetch<CPL>::N : Prefetch<CPL>::N;
    // per-step input: raw cost bytes, or census words (fused variant)
    using RawT = std::conditional_t<FUSED, CensusStep<CPL>, typename Raw<CPL>::T>;

    const int rx = a.rx, ry = a.ry;
    const int W = a.W, H = a.H;
    const int grp = lane / G, q = lane % G;
    const int nslices = KIND == kHoriz ? H : W;
    // Checkpoints: left-to-right walks end with the last column before a
    // segment, right-to-left ones with the first column of segment 1
    constexpr int SEG = RowSegment<G * CPL, LT>::N;
    const int steps = kCkpt ? (rx > 0 ? (W - 1) / SEG * SEG : W - SEG) : (KIND == kHoriz ? W : H);
    if (kCkpt && steps <= 0) {
        if constexpr (SPLIT) split.finish();
        return;
    }
    // groups past the last slice repeat the last slice (identical stores)
    const int jg = min(grp, nslices - 1 - first_slice);

    // Byte planes (largest step penalty <= 255) keep every register value far
    // below 0x7C00, so the minimum of three runs as one packed f16 minimum
    // (vmin3h).  That needs finite stand-ins for "no candidate":
    //   * padded levels d >= D get cost 1023.  Their L stays in [1023, 1278]
    //     and never undercuts a real level: the path minimum m is at most
    //     Cmax <= 64, so m + P2 <= 319 < L(pad) + P1.  (The census-computing
    //     variant, whose planes hold L <= Cmax + P2 <= 255, uses 255.)
    //   * the d - 1 / d + 1 candidate beyond the lane group's ends is 0x0FFF
    //     (OR-ed into a value below 0x1000), above every real candidate.
    //   * P1 is capped at the largest step penalty: a larger P1 never wins
    //     against m + P2 in Eq. 3 (L(d +- 1) >= m), and neither does the cap.
    // 16-bit planes keep saturating u16 arithmetic with 0xFFFF.
    constexpr bool kF16 = sizeof(LT) == 1;
    uint32_t sel[NP];
#pragma unroll
    for (int k = 0; k < NP; ++k)
        sel[k] = FUSED ? pack_selector<CPL>(k, q * CPL, a.D, kF16 ? 0x0C0Du : 0x0D0Du)  // 0x00FF or 0xFFFF
                       : unpack_selector<CPL>(k, q * CPL, a.D, kF16);
    const uint32_t inf = kF16 ? 0x0FFFu : 0xFFFFu;
    const uint32_t edge_lo = q == 0 ? inf << 16 : 0u;  // no d-1 below d = 0
    const uint32_t edge_hi = q == G - 1 ? inf : 0u;    // no d+1 above Dp-1
    const uint32_t P1c = kF16 ? (uint32_t)(ADAPT ? a.P1 : min(a.P1, a.P2)) : (uint32_t)a.P1;
    const u16x2 P1v = as2(P1c * 0x10001u), P2v = as2((uint32_t)a.P2 * 0x10001u);

    const uint32_t plane_bytes = (uint32_t)a.plane;  // cost plane, u8
    const __amdgpu_buffer_rsrc_t rc = buffer_rsrc(a.cost, FUSED ? 0u : plane_bytes);
    // the match buffer starts kCensusGuard words early: a lane's window of
    // CPL words may begin left of column 0 (those words are never used)
    const uint32_t census_bytes = 8u * (uint32_t)W * (uint32_t)H;
    const __amdgpu_buffer_rsrc_t rcl = buffer_rsrc(a.census_l, FUSED ? census_bytes : 0u);
    const __amdgpu_buffer_rsrc_t rcr =
        buffer_rsrc(a.census_r - kCensusGuard, FUSED ? census_bytes + 8u * kCensusGuard : 0u);
    const __amdgpu_buffer_rsrc_t rl = buffer_rsrc(a.lplane, plane_bytes * (uint32_t)sizeof(LT));
    const __amdgpu_buffer_rsrc_t rim = buffer_rsrc(a.img, ADAPT ? (uint32_t)W * (uint32_t)H : 0u);

    // Group 0's position along its slice: pixel index, column (diagonals:
    // kept in [0, W)) and step.  It is the same for the whole wavefront (a
    // scalar); a lane adds its group's distance jl (pixels) from group 0 and
    // its disparities: rows below (horizontal) or columns to the right, less
    // W once a diagonal's group has wrapped to the left border.
    struct Pos {
        int pix, x, t;
    };
    const int pstep = KIND == kHoriz ? rx : ry * W + (KIND == kDiag ? rx : 0);
    Pos cur;
    // a right-to-left walk with checkpoints starts so that its blocks end at
    // multiples of PF and SEG: its first steps (t < 0) repeat the first column
    // and the path starts after them, at t = 0 (step_at_cur; the block that
    // holds t = 0 takes the general form, also where it is the block's first
    // step, as after a lead-in of a whole block)
    constexpr int kAlign = PF > SEG ? PF : SEG;
    const int t_first = kCkpt && rx < 0 ? -((kAlign - W % kAlign) % kAlign) : 0;
    // the wavefront's segment: whole blocks [t_begin, seg_end) of the slice
    int t_begin = t_first, seg_len = 0, seg_end = steps;
    if constexpr (SPLIT) {
        if (split.S > 1) {
            const int blocks = (steps - t_first + kAlign - 1) / kAlign;
            seg_len = (blocks + split.S - 1) / split.S * kAlign;
            t_begin = t_first + split.seg * seg_len;
            seg_end = t_begin + seg_len;
            if (t_begin >= steps) {
                split.finish();
                return;
            }
        }
    }
    cur.t = t_begin;
    const int t_pos = max(t_begin, 0);
    cur.x = KIND == kHoriz ? (rx > 0 ? t_pos : W - 1 - t_pos) : first_slice;
    cur.pix = KIND == kHoriz ? first_slice * W + cur.x : (ry > 0 ? t_pos : H - 1 - t_pos) * W + cur.x;
    // a position stays on the slice's last step, so the lookahead never
    // leaves the slice
    auto advance = [&](Pos& p) {
        const bool more = p.t + 1 < steps && (!kCkpt || p.t >= 0);
        p.t += 1;
        p.pix += more ? pstep : 0;
        if constexpr (KIND == kHoriz) p.x += more ? rx : 0;
        if constexpr (KIND == kDiag) {
            p.x += more ? rx : 0;
            const int wrap = p.x < 0 ? W : (p.x >= W ? -W : 0);
            p.x += wrap;
            p.pix += wrap;
        }
    };
    const int jl0 = KIND == kHoriz ? jg * W : jg;
    const int qofs = q * CPL;
    auto lane_px = [&](const Pos& p) -> int {
        if constexpr (KIND == kDiag) return p.x + jg >= W ? jg - W : jg;
        return jl0;
    };
    // restart column of a diagonal group: where it crosses the side border
    const int border = rx > 0 ? 0 : W - 1;

    // Path state: R = min(L(d), L(d +- 1) + P1) of the last step and the
    // path minimum mm = min_d L(d).  A path start is R = 0, mm = 0.
    u16x2 R[NP];
#pragma unroll
    for (int k = 0; k < NP; ++k) R[k] = as2(0u);
    u16x2 mm = as2(0u);

    // ADAPT: the P2 of a block's PF steps, one step per lane of a row of 16
    // (twice in a u16 pair), each broadcast to its row when its step comes:
    // one load pair and one table lookup per block instead of per step.  The
    // loads run a block ahead, the lookup three steps.  (At a path start R
    // and mm are 0 and the P2 of that step does not matter.)
    uint32_t p2blk = 0, p2next = 0, inten[2] = {0, 0};
    int ax = 0;  // diagonal: the column of the lane's step
    if constexpr (ADAPT && KIND == kDiag) ax = cur.x + jg + rx * (lane & (PF - 1));
    auto adapt_load = [&](int t0) {  // intensities of steps t0 + (lane mod PF) and the one before
        if constexpr (ADAPT) {
            const int t = max(min(t0 + (lane & (PF - 1)), steps - 1), 0);
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const int u = max(t - b, 0);
                uint32_t pix;
                if constexpr (KIND == kHoriz) {
                    pix = (uint32_t)((first_slice + jg) * W + (rx > 0 ? u : W - 1 - u));
                } else {
                    int x = first_slice + jg;
                    if constexpr (KIND == kDiag) {
                        while (ax < 0) ax += W;
                        while (ax >= W) ax -= W;
                        x = ax - b * rx;
                        x += x < 0 ? W : (x >= W ? -W : 0);
                    }
                    pix = (uint32_t)((ry > 0 ? u : H - 1 - u) * W + x);
                }
                inten[b] = __builtin_amdgcn_raw_buffer_load_b8(rim, pix, 0, 0);
            }
            if constexpr (KIND == kDiag) ax += rx * PF;
        }
    };
    auto adapt_lookup = [&] {
        if constexpr (ADAPT) {
            const uint32_t g = inten[0] > inten[1] ? inten[0] - inten[1] : inten[1] - inten[0];
            p2next = a.p2lut[g] * 0x10001u;
        }
    };
    constexpr int kLookupStep = PF - 3;

    // ring[j] holds the raw costs of the step congruent to j modulo PF; the
    // loads lead by PF steps.  c holds the unpacked costs of the current
    // step: a step unpacks the next one's (its load is PF - 1 steps old) and
    // refills its own slot, whose costs the step before unpacked.
    RawT ring[PF];
    u16x2 c[NP];
    auto load_at = [&](const Pos& p) -> RawT {
        const int pix = p.pix + lane_px(p);
        if constexpr (FUSED) {
            RawT cs;
            load_census<CPL>(rcl, rcr, 8u * (uint32_t)pix, 8u * (uint32_t)(pix + kCensusGuard - qofs - (CPL - 1)), cs);
            return cs;
        } else {
            return buffer_load_raw<CPL>(rc, (uint32_t)(pix * Dp + qofs), 0u);
        }
    };
    auto unpack = [&](const RawT& raw, const Pos& p) {
        if constexpr (FUSED) {
            // the lane's disparities are valid (x - d >= 0) for cells
            // c <= x - q*CPL; x of the lane's group is group 0's column + jg
            // (horizontal: same column; diagonal: wrapped)
            const int xg = KIND == kHoriz ? p.x : (KIND == kDiag && p.x + jg >= W ? p.x + jg - W : p.x + jg);
            const int valid_c = xg - q * CPL;
            // smallest column any group of the wavefront is at (uniform): when
            // it is >= Dp - 1, every lane's disparities are valid
            const int xmin_all = KIND == kDiag && p.x + 64 / G - 1 >= W ? 0 : p.x;
            if (xmin_all >= Dp - 1)
                census_costs<CPL, true>(raw, valid_c, (uint32_t)a.cmax, sel, c);
            else
                census_costs<CPL, false>(raw, valid_c, (uint32_t)a.cmax, sel, c);
        } else {
            unpack_costs<CPL>(raw, sel, c);
        }
    };

    // One step: L = C + min(R - mm, P2) (Eq. 3 with the minimum over the
    // path taken out), then R and mm of the next step, side by side, and the
    // unpacking of its costs (`next`, at position `pn`).  `store` puts L
    // where it goes.
    //
    // A wavefront alone on its SIMD issues one instruction every four cycles
    // and an instruction that waits for the previous one's result takes about
    // ten, so a step costs its instruction count or its chain (the minimum
    // over L, then subtract, minimum, add), whichever is longer.  R, the
    // unpacking, the store and the load fill the gaps of the minimum's
    // reduction: the barrier to the compiler's scheduler at the end of a step
    // keeps them there (without it the unpacks of many steps were gathered
    // at the top of a block, where they waited for loads just issued).
    // `store` gets E = L - C (L for the census-computing variant).
    auto step = [&](const RawT& next, const Pos& pn, int j, auto&& store) {
        auto fence = [] { __builtin_amdgcn_sched_barrier(0); };
        u16x2 p2v = P2v;
        if constexpr (ADAPT) {
            p2v = as2(row_broadcast(p2blk, j));
            fence();
        }
        u16x2 L[NP], E[NP];
#pragma unroll
        for (int k = 0; k < NP; ++k) E[k] = R[k] - mm;
        fence();
#pragma unroll
        for (int k = 0; k < NP; ++k) E[k] = vmin(E[k], p2v);
        fence();
#pragma unroll
        for (int k = 0; k < NP; ++k) L[k] = kF16 ? E[k] + c[k] : vadds(E[k], c[k]);
        fence();
        // minimum over the lane's cells, replicated in both halves
        u16x2 tm;
        u16x2 lp[NP];
        auto add_p1 = [&] {
            fence();
#pragma unroll
            for (int k = 0; k < NP; ++k) lp[k] = kF16 ? L[k] + P1v : vadds(L[k], P1v);
            fence();
        };
        if constexpr (kF16 && NP >= 4) {
            u16x2 t = vmin3h(L[0], L[1], L[2]);
            add_p1();
#pragma unroll
            for (int k = 3; k + 1 < NP; k += 2) t = vmin3h(t, L[k], L[k + 1]);
            if constexpr (NP % 2 == 0) t = vmin(t, L[NP - 1]);
            fence();
            unpack(next, pn);
            fence();
            tm = vmin(t, t.yx);
        } else {
            u16x2 t[NP];
#pragma unroll
            for (int k = 0; k < NP; ++k) t[k] = L[k];
#pragma unroll
            for (int w = 1; w < NP; w *= 2)
#pragma unroll
                for (int k = 0; k + w < NP; k += 2 * w) t[k] = vmin(t[k], t[k + w]);
            add_p1();
            tm = vmin(t[0], t[0].yx);
            fence();
            unpack(next, pn);
        }
        uint32_t prev, nxt;
        u16x2 lo0, hiN;
        auto fill = [&](auto stage) {
            constexpr int I = decltype(stage)::value;
            fence();
            if constexpr (I == 0) {
                prev = from_lower<G>(as1(lp[NP - 1])) | edge_lo;
                nxt = from_upper<G>(as1(lp[0])) | edge_hi;
            } else if constexpr (I == 1) {
                lo0 = as2(__builtin_amdgcn_alignbit(as1(lp[NP - 1]), prev, 16));
                hiN = as2(__builtin_amdgcn_alignbit(nxt, as1(lp[0]), 16));
            } else if constexpr (I == 2) {
                store(FUSED ? L : E);
            } else {
#pragma unroll
                for (int k = 0; k < NP; ++k) {
                    const u16x2 lo = k == 0 ? lo0 : lp[k - 1];
                    const u16x2 hi = k == NP - 1 ? hiN : lp[k + 1];
                    R[k] = kF16 ? vmin3h(lo, hi, L[k]) : vmin(vmin(lo, hi), L[k]);
                }
            }
            fence();
        };
        mm = as2(group_min<G>(as1(tm), fill));
    };
    int k = t_begin;  // step of the block's slot 0
    typename Raw<CPL>::T e_last{};  // segments: what the block's last step stored
    // whether slot j of the block is a column the row kernel starts from
    auto at_checkpoint = [&](int j) -> bool {
        if constexpr (PF >= SEG) return (j + 1) % SEG == 0;
        return (j + 1) % PF == 0 && (k - t_first + PF) % SEG == 0;
    };
    // a step at `cur` in the general form (restarts, wraps, any position)
    auto step_at_cur = [&](const RawT& next, int j, auto fix) {
        if constexpr (KIND == kDiag) {
            const int xl = cur.x + jg >= W ? cur.x + jg - W : cur.x + jg;
            if (xl == border) {
#pragma unroll
                for (int k = 0; k < NP; ++k) R[k] = as2(0u);
                mm = as2(0u);
            }
        }
        if constexpr (kCkpt) {
            if (cur.t == 0) {
#pragma unroll
                for (int k = 0; k < NP; ++k) R[k] = as2(0u);
                mm = as2(0u);
            }
        }
        const Pos here = cur;
        advance(cur);
        step(next, cur, j, [&](const u16x2 (&L)[NP]) {
            if constexpr (kCkpt) {
                if (!at_checkpoint(j) || here.t < 0) return;
            }
            if constexpr (decltype(fix)::value) {
                if (j == PF - 1) e_last = pack_u8<CPL>(L);
            }
            if constexpr (kToPlane)
                store_l<CPL, LT, NT>(rl, (uint32_t)((here.pix + lane_px(here)) * Dp + qofs) * (uint32_t)sizeof(LT), 0u, L);
            else
                sink->put(here.t, L);
        });
    };

    adapt_load(cur.t);
    adapt_lookup();
    Pos ahead = cur;
    // Dropped stores (an empty buffer) between the first loads, so that a
    // load has as many memory operations behind it here as in the loop: the
    // compiler's wait before a step then fits the loop (PF - 1 loads and
    // stores may be outstanding) instead of this first block.
    const __amdgpu_buffer_rsrc_t rnone = buffer_rsrc(a.lplane, 0u);
#pragma unroll
    for (int j = 0; j < PF; ++j) {
        ring[j] = load_at(ahead);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (kToPlane && !kCkpt) buffer_store<0>(rnone, 0u, 0u, 0u);
        __builtin_amdgcn_sched_barrier(0);
        advance(ahead);
    }
    unpack(ring[0], cur);

    // Up to PF steps with the loads of the PF steps after them, in the general
    // form: any position, the slice's end, restarts and wraps.
    auto chunk_any = [&](auto whole, auto fix) {
        p2blk = p2next;
        adapt_load(k + PF);
#pragma unroll
        for (int j = 0; j < PF; ++j) {
            __builtin_amdgcn_sched_barrier(0);
            if (decltype(whole)::value || k + j < steps) {
                if (j == kLookupStep) adapt_lookup();
                ring[j] = load_at(ahead);
                step_at_cur(ring[(j + 1) % PF], j, fix);
                advance(ahead);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (!kToPlane) sink->chunk_done();
        k += PF;
    };
    // The same for blocks that neither cross a border nor reach the slice's
    // end with their loads.  Loads and stores share their offsets (the
    // plane's resource is shifted back by PF steps): a scalar one that moves
    // by a step (vertical, diagonal) or a block (horizontal, whose steps
    // differ in the lane offset).
    const uint32_t voff = (uint32_t)(jl0 * Dp + qofs);
    const __amdgpu_buffer_rsrc_t rls = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t*>(reinterpret_cast<const uint8_t*>(a.lplane)) - (ptrdiff_t)PF * pstep * Dp * (int)sizeof(LT), 0,
        -1, 0x00020000);
    uint32_t vstep[KIND == kHoriz ? PF : 1];
#pragma unroll
    for (int j = 0; j < (KIND == kHoriz ? PF : 1); ++j)
        vstep[j] = voff + (uint32_t)((KIND == kHoriz ? (rx > 0 ? j : PF - 1 - j) : 0) * Dp);
    auto chunk_fast = [&](auto fix) {
        if constexpr (!FUSED) {
            uint32_t so = (uint32_t)((ahead.pix - (KIND == kHoriz && rx < 0 ? PF - 1 : 0)) * Dp);
            const uint32_t sstep = (uint32_t)(pstep * Dp);
            p2blk = p2next;
            adapt_load(k + PF);
#pragma unroll
            for (int j = 0; j < PF; ++j) {
                const uint32_t vo = vstep[KIND == kHoriz ? j : 0];
                __builtin_amdgcn_sched_barrier(0);
                if (j == kLookupStep) adapt_lookup();
                ring[j] = buffer_load_raw<CPL>(rc, vo, so);
                step(ring[(j + 1) % PF], cur, j, [&](const u16x2 (&L)[NP]) {
                    if (kCkpt && !at_checkpoint(j)) return;
                    if constexpr (decltype(fix)::value) {
                        if (j == PF - 1) e_last = pack_u8<CPL>(L);
                    }
                    if constexpr (kToPlane)
                        store_l<CPL, LT, NT>(rls, vo * (uint32_t)sizeof(LT), so * (uint32_t)sizeof(LT), L);
                    else
                        sink->put(cur.t + j, L);
                });
                if constexpr (KIND != kHoriz) so += sstep;
            }
            __builtin_amdgcn_sched_barrier(0);
            for (Pos* p : {&cur, &ahead}) {
                p->t += PF;
                p->pix += PF * pstep;
                if constexpr (KIND != kVert) p->x += PF * rx;
                if constexpr (KIND == kDiag) {
                    const int wrap = p->x < 0 ? W : (p->x >= W ? -W : 0);
                    p->x += wrap;
                    p->pix += wrap;
                }
            }
            if constexpr (!kToPlane) sink->chunk_done();
            k += PF;
        }
    };
    // Whole blocks of [k, end): runs of inner ones, and the ones around a
    // diagonal's border crossing or before the slice's end in the general form.
    // With `fixing`, stops after a block whose last step stored what was there.
    auto blocks_to = [&](int end, auto fix) -> bool {
        constexpr bool fixing = decltype(fix)::value;
        bool agreed = false;
        typename Raw<CPL>::T e_old{};
        auto before = [&] {
            if constexpr (fixing) {
                // the block's last step; device scope: past this CU's cache,
                // which may hold the line from before another wavefront stored it
                const uint32_t ofs = (uint32_t)((cur.pix + (PF - 1) * pstep + jl0) * Dp + qofs);
                if constexpr (CPL == 2) {
                    e_old = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rl, ofs, 0, 16);
                } else if constexpr (CPL == 4) {
                    e_old = __builtin_amdgcn_raw_buffer_load_b32(rl, ofs, 0, 16);
                } else if constexpr (CPL == 8) {
                    const auto v = __builtin_amdgcn_raw_buffer_load_b64(rl, ofs, 0, 16);
                    e_old = make_uint2(v[0], v[1]);
                } else {
                    const auto v = __builtin_amdgcn_raw_buffer_load_b128(rl, ofs, 0, 16);
                    e_old = make_uint4(v[0], v[1], v[2], v[3]);
                }
            }
        };
        auto after = [&] {  // k has moved past the block
            if constexpr (fixing) {
                if (kCkpt && PF < SEG && (k - t_first) % SEG != 0) return;
                bool same;
                if constexpr (CPL <= 4)
                    same = e_old == e_last;
                else if constexpr (CPL == 8)
                    same = e_old.x == e_last.x && e_old.y == e_last.y;
                else
                    same = e_old.x == e_last.x && e_old.y == e_last.y && e_old.z == e_last.z && e_old.w == e_last.w;
                agreed = __builtin_amdgcn_ballot_w64(!same) == 0;
            }
        };
        while (k < end && k + PF <= steps && !agreed) {
            int fast = (min(end, steps) - k) / PF;
            if (k + fast * PF + PF > steps) fast -= 1;
            if constexpr (KIND == kDiag) {
                // no group restarts or wraps, neither in a block nor in the
                // steps it loads: columns 1 .. W - S - 1 for group 0
                constexpr int S = 64 / G;
                const int inner = rx > 0 ? (cur.x >= 1 ? (W - S - cur.x) / PF - 1 : 0) : (cur.x < W - S ? cur.x / PF - 1 : 0);
                fast = min(fast, inner);
            }
            if constexpr (FUSED) fast = 0;
            if (kCkpt && t_first < 0 && k <= 0) fast = 0;
            for (int i = 0; i < fast && !agreed; ++i) {
                before();
                chunk_fast(fix);
                after();
            }
            if (k < end && k + PF <= steps && !agreed) {
                before();
                chunk_any(std::true_type{}, fix);
                after();
            }
        }
        return agreed;
    };
    // The conditional steps of the slice's last, partial block come after the
    // loops: a way back from them would make the compiler wait in the loops
    // for loads that may be recent.
    if constexpr (SPLIT) {
        bool agreed = blocks_to(seg_end, std::false_type{});
        while (!agreed && seg_end < steps) {
            split.next_round();
            seg_end += seg_len;
            agreed = blocks_to(seg_end, std::true_type{});
        }
        if (!agreed && k < steps) chunk_any(std::false_type{}, std::false_type{});
        split.finish();
    } else {
        blocks_to(steps, std::false_type{});
        if (k < steps) chunk_any(std::false_type{}, std::false_type{});
    }
}

// ---------------------------------------------------------------------------
// Sum over directions and winner-take-all (Eq. 4), one block per row.
// Lane = pixel: each lane walks its pixel's disparities in runs of 16, sums
// the planes as packed u16 pairs and forms keys (S << 8) | d with one v_perm
// per cell (padded levels get a 0xFF top byte, so they never win).  The left
// disparity is the smallest key of the pixel.  The right view: pixel x at
// disparity d is right pixel x - d, so every (x, d) offers its key to column
// x - d with an LDS atomic minimum; the lanes of a wavefront hit consecutive
// words, and targets x - d < 0 land in a guard region in front of the row.
// The column's winner is argmin_d S(x + d, d), ties to the smallest d.
// ---------------------------------------------------------------------------
// The post stage (3x3 median of both maps, then the left-right check) of
// one pair, read by post_row.
struct PostArgs {
    const uint16_t* dl;
    const uint16_t* dr;
    uint16_t* out;
    int W, H, median, lrcheck, thr;
    int subpixel = 0;  // dl in 1/16 pixel: the check uses its rounding
};

struct WtaArgs {
    const void* lbuf;
    size_t plane;
    uint16_t* dl;  // left disparity (raw, or the final output)
    uint16_t* dr;  // right disparity or nullptr
    int W, H, D, Dp, nplanes;
    int subpixel = 0;  // dl in 1/16 pixel: parabola vertex through S(d-1), S(d), S(d+1)
    // planes of E = L - C: the cost volume, counted once per path; nullptr
    // when the planes hold L
    const uint8_t* cost = nullptr;
    // The post stage run inside the WTA launch (rowcnt != nullptr): per-row
    // counters (zeroed by the census launch of the same frame), `contrib`
    // blocks writing raw rows per image row (2 when one launch makes D_L and
    // D_R with separate blocks), and the post stage's arguments.
    int* rowcnt = nullptr;
    int contrib = 1;
    PostArgs post{};
};

// floor(num / den) for den > 0
__device__ inline int floor_div(int num, int den) {
    const int q = num / den;
    return (num % den != 0 && num < 0) ? q - 1 : q;
}

constexpr int kWtaGuard = 256;  // >= max disparity

// Left disparity in 1/16 pixel: the vertex of the parabola through va =
// S(d - 1), S(d) and vc = S(d + 1) at the winner's key best = (S(d) << 8) | d,
// rounded half up: f = floor((16 (a - c) + den) / (2 den)), den = a + c - 2b
__device__ inline uint32_t subpixel_q4(uint32_t best, uint32_t va, uint32_t vc, int D) {
    const int d = (int)(best & 0xFF);
    int f = 0;
    if (d > 0 && d < D - 1) {
        const int b = (int)((best >> 8) & 0xFFFFu);
        const int den = (int)va + (int)vc - 2 * b;
        if (den > 0) f = floor_div(16 * ((int)va - (int)vc) + den, 2 * den);
    }
    return (uint32_t)(16 * d + f);
}

// Sums of 16 disparities d0..d0+15 of one pixel over NPL planes as 8 packed
// pairs; pair k holds disparities dpair(k) (see below).  Every plane's load
// is issued before the first add, so a lane has all NPL loads in flight.
// NT: the loads are non-temporal (planes that did not fit the memory-side
// cache are streamed once).
template <bool NT>
__device__ inline uint4 load16(const void* p) {
    typedef unsigned v4 __attribute__((ext_vector_type(4)));
    if constexpr (NT) {
        const v4 t = __builtin_nontemporal_load(reinterpret_cast<const v4*>(p));
        return make_uint4(t.x, t.y, t.z, t.w);
    } else {
        return *reinterpret_cast<const uint4*>(p);
    }
}

template <typename LT, int NPL, bool NT>
__device__ inline void sum16(const LT* base, size_t plane, uint32_t (&S)[8]) {
#pragma unroll
    for (int k = 0; k < 8; ++k) S[k] = 0;
    if constexpr (sizeof(LT) == 1) {
        // bytes b0..b3 of dword i -> pairs (b0, b2) and (b1, b3)
        uint4 q[NPL];
#pragma unroll
        for (int p = 0; p < NPL; ++p) q[p] = load16<NT>(base + plane * p);
#pragma unroll
        for (int p = 0; p < NPL; ++p) {
            const uint32_t w[4] = {q[p].x, q[p].y, q[p].z, q[p].w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                S[2 * i] = as1(as2(S[2 * i]) + as2(__builtin_amdgcn_perm(0u, w[i], 0x0C020C00u)));
                S[2 * i + 1] = as1(as2(S[2 * i + 1]) + as2(__builtin_amdgcn_perm(0u, w[i], 0x0C030C01u)));
            }
        }
    } else {
        // u16 pairs are already (d, d + 1)
        uint4 q[NPL][2];
#pragma unroll
        for (int p = 0; p < NPL; ++p) {
            q[p][0] = load16<NT>(base + plane * p);
            q[p][1] = load16<NT>(base + plane * p + 8);
        }
#pragma unroll
        for (int p = 0; p < NPL; ++p) {
            const uint32_t w[8] = {q[p][0].x, q[p][0].y, q[p][0].z, q[p][0].w,
                                   q[p][1].x, q[p][1].y, q[p][1].z, q[p][1].w};
#pragma unroll
            for (int k = 0; k < 8; ++k) S[k] = as1(as2(S[k]) + as2(w[k]));
        }
    }
}

// Adds n times the 16 cost bytes q to the pairs S of sum16<LT>.
template <typename LT>
__device__ inline void add_costs16(const uint4& q, int n, uint32_t (&S)[8]) {
    const uint32_t w[4] = {q.x, q.y, q.z, q.w};
    const u16x2 nn = as2((uint32_t)n * 0x10001u);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const uint32_t sel = sizeof(LT) == 1 ? ((k & 1) ? 0x0C030C01u : 0x0C020C00u) : ((k & 1) ? 0x0C030C02u : 0x0C010C00u);
        S[k] = as1(as2(S[k]) + as2(__builtin_amdgcn_perm(0u, w[k >> 1], sel)) * nn);
    }
}

// Disparities (relative to the run) held by pair k: u8 planes pair 2i =
// (4i, 4i + 2), pair 2i + 1 = (4i + 1, 4i + 3); u16 planes pair k = (2k, 2k+1).
template <typename LT>
__device__ inline void pair_disps(int k, int& lo, int& hi) {
    if constexpr (sizeof(LT) == 1) {
        lo = 4 * (k >> 1) + (k & 1);
        hi = lo + 2;
    } else {
        lo = 2 * k;
        hi = lo + 1;
    }
}

// Minimum over aligned groups of G consecutive lanes (G = 4, 8 or 16);
// every lane of the group receives it.
__device__ inline uint32_t lanes_min(uint32_t v, int G) {
    v = min(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kDppQuadPerm1032, 0xF, 0xF, true));
    v = min(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kDppQuadPerm2301, 0xF, 0xF, true));
    if (G >= 8) v = min(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kDppRowHalfMirror, 0xF, 0xF, true));
    if (G >= 16) v = min(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kDppRowMirror, 0xF, 0xF, true));
    return v;
}

// The winner-take-all of one lane's 16 disparities d0 .. d0+15 of pixel
// (x, y), given their summed costs S (pairs as pair_disps<LT>): keys
// (S << 8) | d with a 0xFF top byte for padded levels; the pixel's smallest
// key over its G lanes (consecutive, aligned) is D_L (1/16-pixel vertex with
// sub-pixel output); with `right`, every (x, d) offers its key to column
// x - d of the row's right-view keys (LDS, atomic minimum; targets x - d < 0
// land in a guard region in front of the row).  s_out (debug): S u16
// [H][W][D].
template <typename LT>
__device__ inline void wta_cells(const WtaArgs& a, int y, int x, int g, int G, const uint32_t (&S)[8],
                                 uint32_t* keyR, bool right, uint16_t* s_out = nullptr, bool valid = true) {
    right = right && valid;
    if (!valid) s_out = nullptr;
    const int d0 = 16 * g;
    uint32_t best = ~0u;
    // right-view targets x - d0 - 15 .. x - d0 from one base address
    uint32_t* tgt = keyR + (x - d0 - 15);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        int dlo, dhi;
        pair_disps<LT>(k, dlo, dhi);
        const uint32_t dpair = (uint32_t)(d0 + dlo) | ((uint32_t)(d0 + dhi) << 8);
        // key = [d, S.lo16, 0] with a 0xFF top byte for padded levels
        const uint32_t klo = __builtin_amdgcn_perm(S[k], dpair, d0 + dlo < a.D ? 0x0C050400u : 0x0D050400u);
        const uint32_t khi = __builtin_amdgcn_perm(S[k], dpair, d0 + dhi < a.D ? 0x0C070601u : 0x0D070601u);
        best = min(best, min(klo, khi));
        if (right) {
            if (d0 + dlo < a.D) atomicMin(tgt + (15 - dlo), klo);
            if (d0 + dhi < a.D) atomicMin(tgt + (15 - dhi), khi);
        }
        if (s_out) {
            uint16_t* o = s_out + ((size_t)y * a.W + x) * a.D;
            if (d0 + dlo < a.D) o[d0 + dlo] = (uint16_t)(S[k] & 0xFFFFu);
            if (d0 + dhi < a.D) o[d0 + dhi] = (uint16_t)(S[k] >> 16);
        }
    }
    best = lanes_min(best, G);
    const int dbest = (int)(best & 0xFF);
    uint32_t outv = (uint32_t)dbest;
    if (a.subpixel) {
        // S(dbest - 1) and S(dbest + 1) from the lanes holding them
        uint32_t va = ~0u, vc = ~0u;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            int dlo, dhi;
            pair_disps<LT>(k, dlo, dhi);
            const uint32_t slo = S[k] & 0xFFFFu, shi = S[k] >> 16;
            if (d0 + dlo == dbest - 1) va = slo;
            if (d0 + dhi == dbest - 1) va = shi;
            if (d0 + dlo == dbest + 1) vc = slo;
            if (d0 + dhi == dbest + 1) vc = shi;
        }
        outv = subpixel_q4(best, lanes_min(va, G), lanes_min(vc, G), a.D);
    }
    if (g == 0 && valid) a.dl[(size_t)y * a.W + x] = (uint16_t)outv;
}

__device__ inline void wta_fold_post(const WtaArgs& a, int y, uint16_t* rview);

template <typename LT, int NPL, bool NT, bool FOLD>
__device__ inline void wta_row_impl(const WtaArgs& a, int y, uint32_t* keyR_smem) {
    uint32_t* keyR = keyR_smem + kWtaGuard;  // keyR[t], t in [-kWtaGuard, W)
    const bool right = a.dr != nullptr;
    if (right)
        for (int i = threadIdx.x; i < a.W + kWtaGuard; i += blockDim.x) keyR_smem[i] = ~0u;
    __syncthreads();
    const LT* planes = reinterpret_cast<const LT*>(a.lbuf);
    // thread (x, g) takes disparities 16g .. 16g + 15 of pixel x; the G runs
    // of a pixel sit on consecutive lanes, so its loads are contiguous
    const int G = a.Dp >> 4;
    const int gshift = G == 4 ? 2 : (G == 8 ? 3 : 4);
    // planes of L - C: each cell's costs once per plane, loaded with the
    // planes (behind a branch they waited for their own latency after them:
    // 160x120, D = 256, 8 paths 47.1 us a frame, 46.0; 640x480, D = 256, 4 paths
    // with the post stage inside 221, 214); planes of L: no times the first
    // plane's bytes
    const uint8_t* costs = a.cost ? a.cost : reinterpret_cast<const uint8_t*>(planes);
    const int times = a.cost ? NPL : 0;
    for (int i = threadIdx.x; i < a.W * G; i += blockDim.x) {
        const int x = i >> gshift, g = i & (G - 1);
        uint32_t S[8];
        const size_t at = ((size_t)y * a.W + x) * a.Dp + 16 * g;
        const uint4 c = load16<false>(costs + at);
        sum16<LT, NPL, NT>(planes + at, a.plane, S);
        add_costs16<LT>(c, times, S);
        wta_cells<LT>(a, y, x, g, G, S, keyR, right);
    }
    if (right) {
        __syncthreads();
        for (int i = threadIdx.x; i < a.W; i += blockDim.x)
            a.dr[(size_t)y * a.W + i] = (uint16_t)(keyR[i] & 0xFF);
    }
    if constexpr (FOLD) wta_fold_post(a, y, reinterpret_cast<uint16_t*>(keyR_smem));
}

// One row of the WTA; the plane count (2, 4 or 8) is a template constant of
// the row's code, so the plane loads unroll.  NT: non-temporal plane loads,
// for planes that exceed the memory-side cache and were stored
// non-temporally.  FOLD: the post stage runs inside the launch (a.rowcnt
// set; wta_fold_post), a separate instantiation so that the plain kernel
// keeps its registers.
template <typename LT, bool NT = false, bool FOLD = false>
__device__ inline void wta_row(const WtaArgs& a, int y, uint32_t* keyR_smem) {
    if (a.nplanes == 2)
        wta_row_impl<LT, 2, NT, FOLD>(a, y, keyR_smem);
    else if (a.nplanes == 4)
        wta_row_impl<LT, 4, NT, FOLD>(a, y, keyR_smem);
    else
        wta_row_impl<LT, 8, NT, FOLD>(a, y, keyR_smem);
}

// ---------------------------------------------------------------------------
// Final pass: the last path direction fused with the sum over directions and
// the winner-take-all (Sec. 3.3), so that direction's L_r plane is never
// written to memory nor read back.  The fused direction is horizontal
// (right-to-left; left-to-right in the 2-path set): the right-view keys need
// whole rows, and a row is the slice of a horizontal direction.
//
// A block has 4 wavefronts, one per SIMD of its CU, in two roles:
//   * 2 producer waves run the recurrence of Eq. 3 along their rows (G = 64
//     lanes per row, 32 when Dp = 64, so a lane holds CPL = Dp / G = 2 or 4
//     disparities) exactly as aggregate_wave does, but put each step's L
//     values into an LDS ring of two chunks of K steps (K = the cost
//     prefetch depth) instead of a plane, and wait at a block barrier after
//     every chunk.  Each recurrence is a dependent chain issued at one
//     instruction per cycle slot of its SIMD, so no other producer shares
//     that SIMD;
//   * 2 consumer waves take chunk c after the barrier that completes it,
//     while the producers work on chunk c + 1.  A chunk has K * R * Dp / 16
//     (pixel, run of 16 disparities) items, M per consumer lane: each adds
//     the P - 1 planes stored by the aggregation launch and the chunk's L
//     values, and runs wta_cells.  The stored planes do not depend on the
//     producers, so a lane loads its items' plane bytes FinalAhead chunks
//     before it needs them (registers), which keeps the memory latency off
//     the per-chunk barrier interval.
// All waves pass the same number of barriers (one after the right-view key
// initialisation, one per chunk, one at the end), after which the block
// writes the right view of its rows from the LDS keys.
// ---------------------------------------------------------------------------
struct FinalArgs {
    SliceArgs agg;          // the fused direction: cost volume, rx = +-1, ry = 0
    const uint8_t* planes;  // the other P - 1 directions' u8 planes (E = L - C), contiguous
    size_t plane;           // bytes per plane (W * H * Dp)
    WtaArgs wta;            // outputs D_L (dl) and D_R (dr, or nullptr), W, H, D, Dp
    uint16_t* s_out;        // debug: S u16 [H][W][D], or nullptr
};

constexpr int kFinalThreads = 256;  // 2 producer + 2 consumer waves

template <int Dp>
struct FinalLayout {
    static constexpr int G = Dp == 64 ? 32 : 64;  // lanes per row
    static constexpr int CPL = Dp / G;             // disparities per lane: 2 or 4
    static constexpr int K = Prefetch<CPL>::N;     // steps per chunk
    static constexpr int NPROD = 2, NC = 2;        // producer and consumer waves
    static constexpr int RW = 64 / G;              // rows per producer wave
    static constexpr int R = NPROD * RW;           // rows per block
    static constexpr int ITEMS = K * R * (Dp / 16);
    static constexpr int M = ITEMS / (64 * NC);    // items per consumer lane and chunk
    static constexpr int ring_bytes = 2 * K * R * Dp;
    static_assert(M * 64 * NC == ITEMS, "whole items per consumer lane");
};

// Rows per final-pass block and its LDS bytes (ring, then the rows' right-
// view keys).
__host__ __device__ inline int final_rows(int Dp) { return Dp == 64 ? 4 : 2; }
__host__ __device__ inline size_t final_smem_bytes(int Dp, int W, bool right) {
    const int R = final_rows(Dp);
    return (size_t)2 * 16 * R * Dp + (right ? (size_t)4 * R * (W + kWtaGuard) : 0);
}

// Chunks of plane loads (NPL: the stored planes and the cost volume) a consumer
// lane keeps in flight, within about 64 registers: 4 * M * NPL registers per
// chunk.  Two chunks of 4 loads of 2 items fill them (4 paths: 640x480, D = 128
// 139 us, one chunk 153; 1280x720, D = 64 247, 291) but with 128 levels and
// non-temporal planes they cost more than they hide (1280x720 446, 387), and
// with 256 levels and 2 paths they spill.
template <int Dp, int M, int NPL, bool NT>
struct FinalAhead {
    static constexpr int n = (Dp == 64 || (Dp == 128 && !NT) ? 16 : 14) / (M * NPL);
    static constexpr int N = n < 1 ? 1 : (n > 3 ? 3 : n);
};

// A producer's sink: step t's values E of row slot `row` go to
// ring[(t / K) % 2][t % K][row][Dp] as bytes in disparity order.
template <int Dp>
struct LdsRingSink {
    uint8_t* ring;
    int row, q;
    __device__ void put(int t, const u16x2 (&l)[FinalLayout<Dp>::CPL / 2]) {
        using L = FinalLayout<Dp>;
        const int buf = (t / L::K) & 1, j = t % L::K;
        auto* dst = reinterpret_cast<typename Raw<L::CPL>::T*>(ring + ((buf * L::K + j) * L::R + row) * Dp + q * L::CPL);
        *dst = pack_u8<L::CPL>(l);
    }
    __device__ void chunk_done() { __syncthreads(); }
};

// Consumer item i of chunk c: pixel (x, y) and its run g, or invalid past
// the row's end or the image's last row (the same for the pixel's Dp / 16
// lanes).
template <int Dp>
struct FinalItem {
    int j, row, g, x, y;
    bool valid;
    __device__ FinalItem(const FinalArgs& f, int y0, int c, int i) {
        using L = FinalLayout<Dp>;
        constexpr int Gp = Dp / 16;
        g = i % Gp;
        const int pix = i / Gp;
        j = pix % L::K;
        row = pix / L::K;
        const int t = c * L::K + j;
        y = y0 + row;
        valid = t < f.wta.W && y < f.wta.H;
        x = f.agg.rx < 0 ? f.wta.W - 1 - t : t;
    }
};

// Plane bytes of an item: one range-checked buffer load per plane, with the
// byte offset of an invalid item past the plane's end (the hardware returns
// zeros), so no branch surrounds a load and the loads of later chunks stay
// in flight while earlier ones are used.  NT: non-temporal (planes that
// exceed the memory-side cache).
template <int NPL, bool NT>
__device__ inline void load_planes16(const __amdgpu_buffer_rsrc_t (&rp)[NPL], uint32_t ofs, uint4 (&q)[NPL]) {
#pragma unroll
    for (int p = 0; p < NPL; ++p) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b128(rp[p], ofs, 0, NT ? 2 : 0);
        q[p] = make_uint4(v[0], v[1], v[2], v[3]);
    }
}

template <int Dp>
__device__ inline uint32_t final_item_offset(const FinalArgs& f, const FinalItem<Dp>& it) {
    return it.valid ? (uint32_t)(((size_t)it.y * f.wta.W + it.x) * Dp + 16 * it.g) : 0xFFFFFFF0u;
}

// One item of a chunk: every lane runs it (invalid items only skip the
// stores and key updates inside wta_cells).
// q: the bytes of the NPL stored planes and, last, of the cost volume
template <int Dp, int NPL>
__device__ inline void final_item_finish(const FinalArgs& f, const FinalItem<Dp>& it, int buf, const uint8_t* ring,
                                         uint32_t* keyR, const uint4 (&q)[NPL + 1]) {
    using L = FinalLayout<Dp>;
    uint32_t S[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) S[k] = 0;
    auto add = [&](const uint4& v) {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            S[2 * k] = as1(as2(S[2 * k]) + as2(__builtin_amdgcn_perm(0u, w[k], 0x0C020C00u)));
            S[2 * k + 1] = as1(as2(S[2 * k + 1]) + as2(__builtin_amdgcn_perm(0u, w[k], 0x0C030C01u)));
        }
    };
#pragma unroll
    for (int p = 0; p < NPL; ++p) add(q[p]);
    {
        const uint32_t w[4] = {q[NPL].x, q[NPL].y, q[NPL].z, q[NPL].w};
        const u16x2 nn = as2((uint32_t)(NPL + 1) * 0x10001u);  // every path's L = E + C
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            S[2 * k] = as1(as2(S[2 * k]) + as2(__builtin_amdgcn_perm(0u, w[k], 0x0C020C00u)) * nn);
            S[2 * k + 1] = as1(as2(S[2 * k + 1]) + as2(__builtin_amdgcn_perm(0u, w[k], 0x0C030C01u)) * nn);
        }
    }
    add(*reinterpret_cast<const uint4*>(ring + ((buf * L::K + it.j) * L::R + it.row) * Dp + 16 * it.g));
    const int W = f.wta.W;
    wta_cells<uint8_t>(f.wta, it.y, it.x, it.g, Dp / 16, S, keyR + it.row * (W + kWtaGuard) + kWtaGuard,
                       f.wta.dr != nullptr, f.s_out, it.valid);
}

template <int Dp, int NPL, bool NT>
__device__ inline void final_pass_block(const FinalArgs& f, int blk, uint8_t* smem) {
    using L = FinalLayout<Dp>;
    const int W = f.wta.W, H = f.wta.H;
    const int y0 = blk * L::R;
    uint8_t* ring = smem;
    uint32_t* keyR = reinterpret_cast<uint32_t*>(smem + L::ring_bytes);
    const bool right = f.wta.dr != nullptr;
    const int kpitch = W + kWtaGuard;
    if (right)
        for (int i = threadIdx.x; i < L::R * kpitch; i += blockDim.x) keyR[i] = ~0u;
    __syncthreads();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    if (wave < L::NPROD) {
        // rows y0 + wave * RW .. (a row past the image repeats the last row;
        // the consumers skip it)
        LdsRingSink<Dp> sink{ring, wave * L::RW + lane / L::G, lane % L::G};
        aggregate_wave<L::G, L::CPL, uint8_t, kHoriz, false, false, false, LdsRingSink<Dp>>(
            f.agg, min(y0 + wave * L::RW, H - 1), lane, &sink);
    } else {
        const int ctid = (wave - L::NPROD) * 64 + lane;
        const int nchunks = (W + L::K - 1) / L::K;
        __amdgpu_buffer_rsrc_t rp[NPL + 1];
#pragma unroll
        for (int p = 0; p < NPL; ++p) rp[p] = buffer_rsrc(f.planes + f.plane * p, (uint32_t)f.plane);
        rp[NPL] = buffer_rsrc(f.agg.cost, (uint32_t)f.plane);
        constexpr int A = FinalAhead<Dp, L::M, NPL + 1, NT>::N;
        // plane bytes of the lane's M items of chunks c .. c + A - 1, slot c % A
        uint4 q[A][L::M][NPL + 1];
        auto item = [&](int c, int m) { return FinalItem<Dp>(f, y0, c, ctid + m * 64 * L::NC); };
#pragma unroll
        for (int s = 0; s < A; ++s)
#pragma unroll
            for (int m = 0; m < L::M; ++m) load_planes16<NPL + 1, NT>(rp, final_item_offset<Dp>(f, item(s, m)), q[s][m]);
        auto chunk = [&](int c, uint4 (&qs)[L::M][NPL + 1]) {
            __syncthreads();  // chunk c is in the ring
#pragma unroll
            for (int m = 0; m < L::M; ++m) final_item_finish<Dp, NPL>(f, item(c, m), c & 1, ring, keyR, qs[m]);
#pragma unroll
            for (int m = 0; m < L::M; ++m) load_planes16<NPL + 1, NT>(rp, final_item_offset<Dp>(f, item(c + A, m)), qs[m]);
        };
        int c0 = 0;
        for (; c0 + A <= nchunks; c0 += A) {
#pragma unroll
            for (int s = 0; s < A; ++s) chunk(c0 + s, q[s]);
        }
#pragma unroll
        for (int s = 0; s < A; ++s)
            if (c0 + s < nchunks) chunk(c0 + s, q[s]);  // the same for every consumer wave
    }
    __syncthreads();
    if (right) {
        for (int row = 0; row < L::R && y0 + row < H; ++row)
            for (int i = threadIdx.x; i < W; i += blockDim.x)
                f.wta.dr[(size_t)(y0 + row) * W + i] = (uint16_t)(keyR[row * kpitch + kWtaGuard + i] & 0xFF);
    }
}

// ---------------------------------------------------------------------------
// 3x3 median (clamp-to-edge) of both maps, then the left-right check.
// The median of 9 is the median of (max of row minima, median of row
// medians, min of row maxima) once each row of 3 is sorted.
// ---------------------------------------------------------------------------
__device__ inline void sort3(uint32_t& a, uint32_t& b, uint32_t& c) {
    uint32_t t;
    if (a > b) { t = a; a = b; b = t; }
    if (b > c) { t = b; b = c; c = t; }
    if (a > b) { t = a; a = b; b = t; }
}

__device__ inline uint32_t med3(uint32_t a, uint32_t b, uint32_t c) {
    return max(min(a, b), min(max(a, b), c));
}

__device__ inline uint32_t median9(const uint16_t* img, int W, int H, int x, int y) {
    uint32_t v[3][3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const uint16_t* row = img + (size_t)clampi(y + j - 1, 0, H - 1) * W;
#pragma unroll
        for (int i = 0; i < 3; ++i) v[j][i] = row[clampi(x + i - 1, 0, W - 1)];
        sort3(v[j][0], v[j][1], v[j][2]);
    }
    const uint32_t lo = max(v[0][0], max(v[1][0], v[2][0]));
    const uint32_t mid = med3(v[0][1], v[1][1], v[2][1]);
    const uint32_t hi = min(v[0][2], min(v[1][2], v[2][2]));
    return med3(lo, mid, hi);
}

// One row of the post stage.  Each thread takes 4 columns per pass so that
// the neighbour loads of a pass are in flight together (a 640-wide row is
// one pass of a 256-thread block); the median and check switches are
// template constants, so no branch splits those loads.  With the check on,
// the first pass loads the D_L and D_R neighbourhoods together (72 loads),
// so the two maps' load latencies overlap; the D_R medians of the whole row
// go to LDS before the barrier, and the check after it reads them at x - d.
template <bool LR, bool MED>
__device__ inline void post_row_impl(const PostArgs& a, int y, uint16_t* rview) {
    constexpr int U = 4;
    const int nt = blockDim.x, x0 = threadIdx.x;
    auto med = [&](const uint16_t* img, int x) -> uint32_t {
        if constexpr (MED)
            return median9(img, a.W, a.H, x, y);
        else
            return img[(size_t)y * a.W + x];
    };
    auto finish = [&](int x, int v) {
        if (x >= a.W) return;
        int o = v;
        if constexpr (LR) {
            const int d = a.subpixel ? (v + 8) >> 4 : v;  // integer disparity of the check
            o = kInvalid;
            if (x - d >= 0) {
                const int e = rview[x - d];
                if (abs(d - e) <= a.thr) o = v;
            }
        }
        a.out[(size_t)y * a.W + x] = (uint16_t)o;
    };
    // first pass: columns x0 + u * nt
    uint32_t dv[U], rv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int x = min(x0 + u * nt, a.W - 1);
        dv[u] = med(a.dl, x);
        if constexpr (LR) rv[u] = med(a.dr, x);
    }
    if constexpr (LR) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (x0 + u * nt < a.W) rview[x0 + u * nt] = (uint16_t)rv[u];
        for (int xb = x0 + U * nt; xb < a.W; xb += U * nt) {
#pragma unroll
            for (int u = 0; u < U; ++u) rv[u] = med(a.dr, min(xb + u * nt, a.W - 1));
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (xb + u * nt < a.W) rview[xb + u * nt] = (uint16_t)rv[u];
        }
        __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < U; ++u) finish(x0 + u * nt, (int)dv[u]);
    for (int xb = x0 + U * nt; xb < a.W; xb += U * nt) {
#pragma unroll
        for (int u = 0; u < U; ++u) dv[u] = med(a.dl, min(xb + u * nt, a.W - 1));
#pragma unroll
        for (int u = 0; u < U; ++u) finish(xb + u * nt, (int)dv[u]);
    }
}

__device__ inline void post_row(const PostArgs& a, int y, uint16_t* rview) {
    if (a.lrcheck) {
        if (a.median)
            post_row_impl<true, true>(a, y, rview);
        else
            post_row_impl<true, false>(a, y, rview);
    } else {
        if (a.median)
            post_row_impl<false, true>(a, y, rview);
        else
            post_row_impl<false, false>(a, y, rview);
    }
}

// The post stage inside the WTA launch, without any wait: row r's median
// and check need the raw maps of rows r - 1 .. r + 1, so a block that has
// written its raw row y counts itself into rows y - 1 .. y + 1, and the
// block whose count completes a row (the last of the blocks that write its
// neighbourhood, in whatever order they ran) runs that row's post stage and
// clears its counter.  Every wave waits for its raw-map stores to complete
// (a block barrier alone does not wait for global stores), then one thread
// releases them with a device-scope fence (a write-back of this XCD's L2,
// so one per block, not one per wave) before the counting, and acquires the
// other blocks' rows after it (they may have been written through another
// L2).
__device__ inline void wta_fold_post(const WtaArgs& a, int y, uint16_t* rview) {
    __shared__ int todo[3];
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): expcnt and lgkmcnt left at their maxima
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence();
        __builtin_amdgcn_s_waitcnt(0x0F70);  // the write-back has completed
        for (int k = 0; k < 3; ++k) {
            const int r = y - 1 + k;
            todo[k] = 0;
            if (r < 0 || r >= a.H) continue;
            const int need = a.contrib * ((r > 0) + 1 + (r < a.H - 1));
            if (atomicAdd(&a.rowcnt[r], 1) + 1 == need) {
                atomicExch(&a.rowcnt[r], 0);
                todo[k] = 1;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        __builtin_amdgcn_s_waitcnt(0x0F70);  // the invalidation has completed before the barrier
    }
    __syncthreads();
    for (int k = 0; k < 3; ++k) {
        if (todo[k]) {
            post_row(a.post, y - 1 + k, rview);
            __syncthreads();  // rview is reused by the next row
        }
    }
}


}  // namespace dev
}  // namespace sgm
