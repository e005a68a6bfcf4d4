// The batched aggregation of batches with an adaptive-P2 pair.
#include "sgm_batch_agg_impl.h"

namespace sgm {

void launch_batch_agg_adapt(bool nt, bool ckpt, int blocks, const BatchItem* items, const WorkItem* work, int nquads,
                            unsigned* queue_counter, int P1, int P2, hipStream_t stream) {
    launch_batch_agg_t<true>(nt, ckpt, blocks, items, work, nquads, queue_counter, P1, P2, stream);
}

}  // namespace sgm
