// The batched operator of any degree, single precision.
#include "ax_any.h"

namespace hb {

hb_status launch_batch_any32(const WorkItem *items, int nitems, size_t lds, const BatchProb *probs, hipStream_t s)
{
    return launch_batch_any<float, false>(items, nitems, lds, probs, s);
}

}  // namespace hb
