// Tables of the batched kernels and the launchers of the batched aggregation
// (sgm_batch_agg.hip; sgm_batch_agg_adapt.hip for batches with an adaptive-P2
// pair), compiled as separate sources so that they build in parallel.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace sgm {

// One pair as the batched kernels see it.
struct BatchItem {
    const uint8_t* left;
    const uint8_t* right;
    uint16_t* out;
    uint64_t* census_l;
    uint64_t* census_r;
    uint8_t* cost;
    uint8_t* cost_r;  // right-base costs (lr_full), else nullptr
    void* lbuf;       // L_r planes; with lr_full the right-base planes follow
    uint16_t* dl;
    uint16_t* dr;
    int W, H, D, Dp, P, cmax, l16, median, lrcheck, thr, csct, gh, gv, subpixel, lr_full, adaptive;
    int census_blk0, cost_blk0, wta_blk0, post_blk0;  // first block in each launch (wta_blk0: in
                                                      // the winner-take-all launch or the row
                                                      // launch of its kernel variant)
};

// One aggregation work item: S = 64 / G slices of one direction of one pair;
// rb = 1 for a direction of the right-base SGM (full left-right check);
// item = -1 marks an empty place of a quad.
struct WorkItem {
    int item, plane, rx, ry, first, steps, rb;
};

// Work items go out four at a time, one per wavefront of a workgroup (a
// quad).  Opposite directions over the same pixels share a quad (A, A, B,
// B): the axis-aligned ones over the same two slice groups, the diagonals
// over the groups that cover (most of) the same pixels.  Both walks over a
// pixel's costs then run on one CU and its L2, and the second read can hit
// there, as in the single-pair aggregation launch.
constexpr int kQuad = 4;

// Index of the pair whose block range [blk0, next blk0) holds block b.
template <int BatchItem::*FIRST>
__device__ inline int find_item(const BatchItem* items, int n, int b) {
    int lo = 0, hi = n;  // items[lo].*FIRST <= b < items[hi].*FIRST
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (items[mid].*FIRST <= b)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

// ckpt: the row kernel follows; else the winner-take-all over whole planes.
void launch_batch_agg(bool nt, bool ckpt, int blocks, const BatchItem* items, const WorkItem* work, int nquads,
                      unsigned* queue_counter, int P1, int P2, hipStream_t stream);
void launch_batch_agg_adapt(bool nt, bool ckpt, int blocks, const BatchItem* items, const WorkItem* work, int nquads,
                            unsigned* queue_counter, int P1, int P2, hipStream_t stream);

}  // namespace sgm
