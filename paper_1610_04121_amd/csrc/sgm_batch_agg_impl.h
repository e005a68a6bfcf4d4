// The persistent batched aggregation kernel (included by sgm_batch_agg.hip
// and sgm_batch_agg_adapt.hip).
#pragma once

#include "sgm_batch_agg.h"
#include "sgm_device.h"

namespace sgm {

namespace {

using namespace dev;

// NT: non-temporal L_r stores (the batch's planes exceed the memory-side
// cache); ADAPT: adaptive P2 (the block's penalty table is in s.p2lut); CKPT:
// horizontal directions store what the row kernel needs, else whole planes.
template <typename LT, int Dp, bool NT, bool ADAPT, bool CKPT>
__device__ __attribute__((always_inline)) inline void aggregate_item(const SliceArgs& s, int kind, int g, int first,
                                                                     int lane) {
    if (kind == kHoriz) {
        using Sink = std::conditional_t<CKPT, CkptSink, PlaneSink>;
        if (g == 32)
            aggregate_wave<32, Dp / 32, LT, kHoriz, false, ADAPT, NT, Sink>(s, first, lane);
        else
            aggregate_wave<16, Dp / 16, LT, kHoriz, false, ADAPT, NT, Sink>(s, first, lane);
    } else if (kind == kVert) {
        if (g == 32)
            aggregate_wave<32, Dp / 32, LT, kVert, false, ADAPT, NT>(s, first, lane);
        else
            aggregate_wave<16, Dp / 16, LT, kVert, false, ADAPT, NT>(s, first, lane);
    } else {
        if (g == 32)
            aggregate_wave<32, Dp / 32, LT, kDiag, false, ADAPT, NT>(s, first, lane);
        else
            aggregate_wave<16, Dp / 16, LT, kDiag, false, ADAPT, NT>(s, first, lane);
    }
}

// g: the work item's lanes per slice (its pair's horizontal or other group
// width, by the direction's kind)
template <typename LT, bool NT, bool ADAPT, bool CKPT>
__device__ __attribute__((always_inline)) inline void aggregate_item_dp(const SliceArgs& s, int Dp, int kind, int g,
                                                                        int first, int lane) {
    if (Dp == 64)
        aggregate_item<LT, 64, NT, ADAPT, CKPT>(s, kind, g, first, lane);
    else if (Dp == 128)
        aggregate_item<LT, 128, NT, ADAPT, CKPT>(s, kind, g, first, lane);
    else
        aggregate_item<LT, 256, NT, ADAPT, CKPT>(s, kind, g, first, lane);
}

// ANY_ADAPT: some pair of the batch uses the adaptive P2 (a second
// instantiation, so batches without one keep the smaller kernel).  A
// workgroup takes one quad of work items at a time, wavefront k its item k;
// the quad's items have the same length, so its wavefronts finish together.
template <bool NT, bool ANY_ADAPT, bool CKPT>
__global__ __launch_bounds__(256) void aggregate_batch_kernel(const BatchItem* items, const WorkItem* work,
                                                              int nquads, unsigned* queue_counter, int P1, int P2) {
    __shared__ uint16_t p2lut[ANY_ADAPT ? 256 : 1];
    __shared__ unsigned quad;
    __shared__ uint16_t p2const[ANY_ADAPT ? 256 : 1];
    if constexpr (ANY_ADAPT) {  // P1, P2 belong to the batch: one table per block
        fill_p2_lut(p2lut, P1, P2);
        p2const[threadIdx.x] = (uint16_t)P2;
    }
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    for (;;) {
        // the barrier also ends every wavefront's read of the previous quad
        // index (and, on the first pass, the penalty table's fill)
        __syncthreads();
        if (threadIdx.x == 0) quad = atomicAdd(queue_counter, 1u);
        __syncthreads();
        const unsigned q = __builtin_amdgcn_readfirstlane(quad);
        if (q >= (unsigned)nquads) break;
        const WorkItem w = work[(size_t)q * kQuad + wave];
        if (w.item < 0) continue;
        const BatchItem& it = items[w.item];
        const uint32_t plane = (uint32_t)it.W * (uint32_t)it.H * (uint32_t)it.Dp;
        void* lplane = it.l16 ? (void*)(reinterpret_cast<uint16_t*>(it.lbuf) + (size_t)plane * w.plane)
                              : (void*)(reinterpret_cast<uint8_t*>(it.lbuf) + (size_t)plane * w.plane);
        // a right-base direction reads the right-base costs; the adaptive P2
        // follows its SGM's base image
        SliceArgs s{w.rb ? it.cost_r : it.cost, it.census_l, it.census_r, lplane, plane, it.W, it.H, it.D, P1, P2,
                    it.cmax, w.rx, w.ry};
        s.img = w.rb ? it.right : it.left;
        s.p2lut = ANY_ADAPT ? p2lut : nullptr;
        const int kind = w.ry == 0 ? kHoriz : (w.rx == 0 ? kVert : kDiag);
        const int g = kind == kHoriz ? it.gh : it.gv;
        // in a batch with an adaptive-P2 pair the others take the same code
        // with a table of their constant P2 (and, as without it, P1 capped at
        // the largest penalty of a step on byte planes)
        if constexpr (ANY_ADAPT) {
            if (!it.adaptive) {
                s.p2lut = p2const;
                if (!it.l16) s.P1 = min(P1, P2);
            }
        }
        if (it.l16)
            aggregate_item_dp<uint16_t, NT, ANY_ADAPT, CKPT>(s, it.Dp, kind, g, w.first, lane);
        else
            aggregate_item_dp<uint8_t, NT, ANY_ADAPT, CKPT>(s, it.Dp, kind, g, w.first, lane);
    }
}

template <bool ANY_ADAPT>
void launch_batch_agg_t(bool nt, bool ckpt, int blocks, const BatchItem* items, const WorkItem* work, int nquads,
                        unsigned* queue_counter, int P1, int P2, hipStream_t stream) {
    auto k = ckpt ? (nt ? aggregate_batch_kernel<true, ANY_ADAPT, true> : aggregate_batch_kernel<false, ANY_ADAPT, true>)
                  : (nt ? aggregate_batch_kernel<true, ANY_ADAPT, false> : aggregate_batch_kernel<false, ANY_ADAPT, false>);
    hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(256), 0, stream, items, work, nquads, queue_counter, P1, P2);
}

}  // namespace

}  // namespace sgm
