// The batched operator of any degree, double precision, masked.
#include "ax_any.h"

namespace hb {

hb_status launch_batch_any64_d(const WorkItem *items, int nitems, size_t lds, const BatchProb *probs, hipStream_t s)
{
    return launch_batch_any<double, true>(items, nitems, lds, probs, s);
}

}  // namespace hb
