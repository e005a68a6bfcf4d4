// Launchers of the row kernel (sgm_row_device.h), one source per padded
// disparity range (sgm_row_64.hip, sgm_row_128.hip, sgm_row_256.hip) so that
// they build in parallel.
#pragma once

#include <hip/hip_runtime.h>

#include "sgm_batch_agg.h"
#include "sgm_row_device.h"

namespace sgm {

// Which instantiation of the row kernel to launch.
struct RowVariant {
    int n_paths;
    bool l16;   // 16-bit planes
    bool nt;    // planes loaded non-temporally
    bool pair;  // two values fit a byte together
    bool sub;   // sub-pixel output
};

// One launch: the rows of one SGM (l), of two (l, then r: the full left-right
// check; r.cost set), or, with n > 0, of the batch pairs items[0 .. n) (all of
// this variant), blocks 0 .. being their rows in order of wta_blk0.
struct RowLaunch {
    dev::RowArgs l, r;
    const BatchItem* items;
    int n, P1, P2;  // batch: pairs and penalties
};

hipError_t launch_row_64(const RowLaunch& a, const RowVariant& v, int blocks, int waves, size_t smem, hipStream_t stream);
hipError_t launch_row_128(const RowLaunch& a, const RowVariant& v, int blocks, int waves, size_t smem, hipStream_t stream);
hipError_t launch_row_256(const RowLaunch& a, const RowVariant& v, int blocks, int waves, size_t smem, hipStream_t stream);

// Wavefronts of a row's workgroup: a wavefront takes 4 segments at a time (2
// with 256 levels).  8 wavefronts put two on each SIMD of a CU; 5 or 7 leave
// SIMDs unequally loaded (1242x375, D = 128, 8 paths, whole call: 275, 265 and
// 260 us with 5, 7 and 8).
inline int row_waves(int W, int Dp, bool l16) {
    const int cols = (Dp == 256 ? 2 : 4) * (l16 ? 8 : 16);
    const int units = (W + cols - 1) / cols;
    return units < 8 ? units : 8;
}

}  // namespace sgm
