// The row kernel of pairs padded to 64 disparity levels.
#include "sgm_row_impl.h"

namespace sgm {

hipError_t launch_row_64(const RowLaunch& a, const RowVariant& v, int blocks, int waves, size_t smem, hipStream_t stream) {
    return launch_row_dp<64>(a, v, blocks, waves, smem, stream);
}

}  // namespace sgm
