// The aggregation kernel of one padded disparity range and its launcher
// (included by sgm_agg_64.hip, sgm_agg_128.hip and sgm_agg_256.hip).
#pragma once

#include "sgm_agg.h"

namespace sgm {

namespace {

using namespace dev;

// One launch covers every direction.  Horizontal slices (the longest when
// W > H) may use a different group width than the others, so that the longest
// dependency chains get the fewest instructions per step.  SPLIT: slices in
// segments (dev::Split), an instantiation of its own because the walk that can
// stop early is scheduled worse where nothing is split (640x480, D = 128,
// 4 paths: 100.0 us per call against 98.8).
template <int Dp, typename LT, bool FUSED, bool ADAPT, bool NT, bool SPLIT>
__global__ __launch_bounds__(256) void aggregate_kernel(AggArgs a) {
    __shared__ uint16_t p2lut[ADAPT ? 256 : 1];
    if constexpr (ADAPT) {  // every wave of the block takes part before any leaves
        fill_p2_lut(p2lut, a.base.P1, a.base.P2);
        __syncthreads();
    }
    __shared__ int open[SPLIT ? 4 : 1];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
    // the wavefront's slice group and, with split groups, its segment of it
    Split split;
    int unit = wave;
    if constexpr (SPLIT) {
        unit = wave >> (a.split == 2 ? 1 : 2);
        split = Split{wave & (a.split - 1), a.split, open, wave & 3};
    }
    if (unit >= a.total) {
        if constexpr (SPLIT) split.finish();
        return;
    }
    int r = 0;
    while (r + 1 < a.ndirs && unit >= a.start[r + 1]) ++r;
    int local = unit - a.start[r];
    // The 2n waves of a pair of opposite directions over the same n slice
    // groups interleave two by two (A, A, B, B per workgroup; A, B when each
    // takes two wavefronts), so both directions' waves over the same slices
    // share a CU and its L2: the second read of a slice's costs can hit where
    // the two walks pass close in time.  A bijection between the pair's waves
    // and (direction, slice group); an odd n ends with one wave of each.
    const int r0 = (r > 0 && a.paired[r - 1]) ? r - 1 : r;
    if (a.paired[r0]) {
        const int n = a.start[r0 + 1] - a.start[r0];
        const int j = unit - a.start[r0];
        const int g = j >> 2, w4 = j & 3;
        if (!SPLIT && 4 * g + 4 <= 2 * n) {
            r = r0 + (w4 >> 1);
            local = 2 * g + (w4 & 1);
        } else {
            r = r0 + (j & 1);
            local = j >> 1;
        }
    }
    SliceArgs s = a.base;
    s.rx = a.rx[r];
    s.ry = a.ry[r];
    s.cost = a.cost[r];
    s.img = a.img[r];
    s.p2lut = ADAPT ? p2lut : nullptr;
    s.lplane = reinterpret_cast<LT*>(a.lbuf) + (size_t)s.plane * a.plane_index[r];
    auto walk = [&](auto lanes, auto kind) {
        constexpr int G = decltype(lanes)::value, KIND = decltype(kind)::value;
        const int first = local * (64 / G);
        if constexpr (KIND == kHoriz && !FUSED) {
            if (a.ckpt) {
                aggregate_wave<G, Dp / G, LT, KIND, FUSED, ADAPT, NT, CkptSink, SPLIT>(s, first, lane, nullptr, split);
                return;
            }
        }
        aggregate_wave<G, Dp / G, LT, KIND, FUSED, ADAPT, NT, PlaneSink, SPLIT>(s, first, lane, nullptr, split);
    };
    using std::integral_constant;
    if (s.ry == 0) {
        const integral_constant<int, kHoriz> kind;
        if constexpr (Dp >= 128) {  // 64 lanes need at least 2 levels per lane
            if (a.gh == 64) {
                walk(integral_constant<int, 64>{}, kind);
                return;
            }
        }
        if (a.gh == 32)
            walk(integral_constant<int, 32>{}, kind);
        else
            walk(integral_constant<int, 16>{}, kind);
    } else if (s.rx == 0) {
        const integral_constant<int, kVert> kind;
        if (a.gv == 32)
            walk(integral_constant<int, 32>{}, kind);
        else
            walk(integral_constant<int, 16>{}, kind);
    } else if constexpr (!SPLIT) {  // (only path sets without diagonals are split)
        const integral_constant<int, kDiag> kind;
        if (a.gv == 32)
            walk(integral_constant<int, 32>{}, kind);
        else
            walk(integral_constant<int, 16>{}, kind);
    }
}

template <int Dp, typename LT, bool FUSED, bool ADAPT, bool NT, bool SPLIT = false>
hipError_t launch_agg_t(const AggArgs& a, hipStream_t stream) {
    hipLaunchKernelGGL((aggregate_kernel<Dp, LT, FUSED, ADAPT, NT, SPLIT>), dim3((a.total * a.split + 3) / 4),
                       dim3(256), 0, stream, a);
    return hipGetLastError();
}

template <int Dp, typename LT>
hipError_t launch_agg_lt(const AggArgs& a, const AggVariant& v, hipStream_t stream) {
    if constexpr (sizeof(LT) == 1) {
        // (the rounds read back what the walk stored: no non-temporal stores)
        if (a.split > 1 && v.adaptive) return launch_agg_t<Dp, LT, false, true, false, true>(a, stream);
        if (a.split > 1) return launch_agg_t<Dp, LT, false, false, false, true>(a, stream);
    }
    if (v.adaptive) return launch_agg_t<Dp, LT, false, true, false>(a, stream);
    if (v.fused) return launch_agg_t<Dp, LT, true, false, false>(a, stream);
    if (v.nt) return launch_agg_t<Dp, LT, false, false, true>(a, stream);
    return launch_agg_t<Dp, LT, false, false, false>(a, stream);
}

template <int Dp>
hipError_t launch_agg_dp(const AggArgs& a, const AggVariant& v, hipStream_t stream) {
    return v.l16 ? launch_agg_lt<Dp, uint16_t>(a, v, stream) : launch_agg_lt<Dp, uint8_t>(a, v, stream);
}

}  // namespace

}  // namespace sgm
