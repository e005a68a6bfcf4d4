// The row kernel of pairs padded to 128 disparity levels.
#include "sgm_row_impl.h"

namespace sgm {

hipError_t launch_row_128(const RowLaunch& a, const RowVariant& v, int blocks, int waves, size_t smem, hipStream_t stream) {
    return launch_row_dp<128>(a, v, blocks, waves, smem, stream);
}

}  // namespace sgm
