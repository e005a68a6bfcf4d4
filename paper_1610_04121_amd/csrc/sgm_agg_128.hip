// The aggregation launch of pairs padded to 128 disparity levels.
#include "sgm_agg_impl.h"

namespace sgm {

hipError_t launch_agg_128(const AggArgs& a, const AggVariant& v, hipStream_t stream) {
    return launch_agg_dp<128>(a, v, stream);
}

}  // namespace sgm
