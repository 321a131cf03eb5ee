// The batched operator of any degree, single precision, masked.
#include "ax_any.h"

namespace hb {

hb_status launch_batch_any32_d(const WorkItem *items, int nitems, size_t lds, const BatchProb *probs, hipStream_t s)
{
    return launch_batch_any<float, true>(items, nitems, lds, probs, s);
}

}  // namespace hb
