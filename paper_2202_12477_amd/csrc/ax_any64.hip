// The batched operator of any degree, double precision.
#include "ax_any.h"

namespace hb {

namespace {

template <int N>
size_t lds_of(int n, int v, bool fp32)
{
    if constexpr (N == 0) {
        return 0;
    } else {
        if (n != N) return lds_of<N - 1>(n, v, fp32);
        return (fp32 ? 4 : 8) * static_cast<size_t>(v == 1 ? Shape<N, 1>::lds : Shape<N, 0>::lds);
    }
}

}  // namespace

size_t batch_ax_lds(int N, int variant, bool fp32) { return lds_of<kMaxN>(N, variant, fp32); }

hb_status launch_batch_any64(const WorkItem *items, int nitems, size_t lds, const BatchProb *probs, hipStream_t s)
{
    return launch_batch_any<double, false>(items, nitems, lds, probs, s);
}

}  // namespace hb
