// The aggregation kernel of one padded disparity range and its launcher
// (included by sgm_agg_64.hip, sgm_agg_128.hip and sgm_agg_256.hip).
#pragma once

#include "sgm_agg.h"

namespace sgm {

namespace {

using namespace dev;

// One launch covers every direction.  Horizontal slices (the longest when
// W > H) may use a different group width GH than the others (GV), so that
// the longest dependency chains get the fewest instructions per step.
template <int GH, int GV, int Dp, typename LT, bool FUSED, bool ADAPT, bool NT>
__global__ __launch_bounds__(256) void aggregate_kernel(AggArgs a) {
    __shared__ uint16_t p2lut[ADAPT ? 256 : 1];
    if constexpr (ADAPT) {  // every wave of the block takes part before any leaves
        fill_p2_lut(p2lut, a.base.P1, a.base.P2);
        __syncthreads();
    }
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
    if (wave >= a.total) return;
    int r = 0;
    while (r + 1 < a.ndirs && wave >= a.start[r + 1]) ++r;
    int local = wave - a.start[r];
    // The 2n waves of a pair of opposite directions over the same n slice
    // groups interleave two by two (A, A, B, B per workgroup), so both
    // directions' waves over the same slices share a CU and its L2: the
    // second read of a slice's costs can hit where the two walks pass close
    // in time.  A bijection between the pair's waves and (direction, slice
    // group); an odd n ends with one wave of each.
    const int r0 = (r > 0 && a.paired[r - 1]) ? r - 1 : r;
    if (a.paired[r0]) {
        const int n = a.start[r0 + 1] - a.start[r0];
        const int j = wave - a.start[r0];
        const int g = j >> 2, w4 = j & 3;
        if (4 * g + 4 <= 2 * n) {
            r = r0 + (w4 >> 1);
            local = 2 * g + (w4 & 1);
        } else {
            r = r0 + (w4 & 1);
            local = 2 * g;
        }
    }
    SliceArgs s = a.base;
    s.rx = a.rx[r];
    s.ry = a.ry[r];
    s.cost = a.cost[r];
    s.img = a.img[r];
    s.p2lut = ADAPT ? p2lut : nullptr;
    s.lplane = reinterpret_cast<LT*>(a.lbuf) + (size_t)s.plane * a.plane_index[r];
    if (s.ry == 0) {
        if constexpr (!FUSED) {
            if (a.ckpt) {
                aggregate_wave<GH, Dp / GH, LT, kHoriz, FUSED, ADAPT, NT, CkptSink>(s, local * (64 / GH), lane);
                return;
            }
        }
        aggregate_wave<GH, Dp / GH, LT, kHoriz, FUSED, ADAPT, NT>(s, local * (64 / GH), lane);
    } else if (s.rx == 0) {
        aggregate_wave<GV, Dp / GV, LT, kVert, FUSED, ADAPT, NT>(s, local * (64 / GV), lane);
    } else {
        aggregate_wave<GV, Dp / GV, LT, kDiag, FUSED, ADAPT, NT>(s, local * (64 / GV), lane);
    }
}

template <int GH, int GV, int Dp, typename LT, bool FUSED, bool ADAPT, bool NT>
hipError_t launch_agg_t(const AggArgs& a, hipStream_t stream) {
    hipLaunchKernelGGL((aggregate_kernel<GH, GV, Dp, LT, FUSED, ADAPT, NT>), dim3((a.total + 3) / 4), dim3(256), 0,
                       stream, a);
    return hipGetLastError();
}

template <int Dp, typename LT, bool FUSED, bool ADAPT, bool NT>
hipError_t launch_agg_lanes(const AggArgs& a, const AggVariant& v, hipStream_t stream) {
    switch (v.gh * 100 + v.gv) {
        case 1616: return launch_agg_t<16, 16, Dp, LT, FUSED, ADAPT, NT>(a, stream);
        case 3216: return launch_agg_t<32, 16, Dp, LT, FUSED, ADAPT, NT>(a, stream);
        case 3232: return launch_agg_t<32, 32, Dp, LT, FUSED, ADAPT, NT>(a, stream);
        default: break;
    }
    if constexpr (Dp >= 128) {  // 64 lanes need at least 2 levels per lane
        if (v.gh == 64 && v.gv == 16) return launch_agg_t<64, 16, Dp, LT, FUSED, ADAPT, NT>(a, stream);
        if (v.gh == 64 && v.gv == 32) return launch_agg_t<64, 32, Dp, LT, FUSED, ADAPT, NT>(a, stream);
    }
    return hipErrorInvalidValue;
}

template <int Dp, typename LT>
hipError_t launch_agg_lt(const AggArgs& a, const AggVariant& v, hipStream_t stream) {
    if (v.adaptive) return launch_agg_lanes<Dp, LT, false, true, false>(a, v, stream);
    if (v.fused) return launch_agg_lanes<Dp, LT, true, false, false>(a, v, stream);
    if (v.nt) return launch_agg_lanes<Dp, LT, false, false, true>(a, v, stream);
    return launch_agg_lanes<Dp, LT, false, false, false>(a, v, stream);
}

template <int Dp>
hipError_t launch_agg_dp(const AggArgs& a, const AggVariant& v, hipStream_t stream) {
    return v.l16 ? launch_agg_lt<Dp, uint16_t>(a, v, stream) : launch_agg_lt<Dp, uint8_t>(a, v, stream);
}

}  // namespace

}  // namespace sgm
