// The single-pair aggregation launch: its argument table and the launchers
// of each padded disparity range, compiled as separate sources
// (sgm_agg_64.hip, sgm_agg_128.hip, sgm_agg_256.hip) so that they build in
// parallel.
#pragma once

#include <hip/hip_runtime.h>

#include "sgm_device.h"

namespace sgm {

// Direction table of one pair's aggregation launch: the directions of one
// SGM, or of two (left-base and right-base, for the full left-right check).
constexpr int kMaxLaunchDirs = 2 * kMaxDirs;
struct AggArgs {
    dev::SliceArgs base;          // shared fields; rx, ry, cost, lplane set per direction
    void* lbuf;              // all L_r planes
    int ndirs, total;
    int start[kMaxLaunchDirs + 1];  // first slice group of each direction
    int rx[kMaxLaunchDirs], ry[kMaxLaunchDirs], plane_index[kMaxLaunchDirs];
    const uint8_t* cost[kMaxLaunchDirs];  // the cost volume each direction reads
    const uint8_t* img[kMaxLaunchDirs];   // its SGM's base image (adaptive P2)
    // paired[k]: directions k and k + 1 are opposite, axis-aligned and have
    // the same wave count; their waves interleave (see aggregate_kernel)
    int paired[kMaxLaunchDirs];
    // the horizontal directions keep only the columns the row kernel enters
    // its segments from (CkptSink)
    int ckpt;
    int gh, gv;  // lanes per horizontal (16, 32, 64) / other (16, 32) slice
    // wavefronts per slice group (1, 2 or 4 segments, dev::Split); start and
    // total count slice groups
    int split;
};

// Which instantiation of the aggregation kernel to launch.
struct AggVariant {
    bool l16, fused, adaptive, nt;
};

hipError_t launch_agg_64(const AggArgs& a, const AggVariant& v, hipStream_t stream);
hipError_t launch_agg_128(const AggArgs& a, const AggVariant& v, hipStream_t stream);
hipError_t launch_agg_256(const AggArgs& a, const AggVariant& v, hipStream_t stream);

}  // namespace sgm
