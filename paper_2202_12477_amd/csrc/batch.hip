// Batched CG over independent problems of different sizes and degrees.
//
// All problems advance together: one iteration is one operator launch over a work
// list of (problem, element tile), or on large batches one per (degree, precision)
// class, then one launch each for the residual and the update over all problems (for
// alpha and beta too where a problem has many partial sums).  Each problem keeps its own device state (CgState), so problems
// at different iterations, or already finished, share the same launches
// (finished ones return at once).  The host rebuilds the work lists only when
// the set of running problems changes.  This file holds the vector and scalar
// steps; the batched operator kernel is instantiated with the single-problem
// operator, per degree range (ax_impl.h, ax_n*.hip), and launched through the
// schedule table (ax.hip).
#include "ax_impl.h"
#include "cg_steps.h"
#include "common.h"
#include "reduce.h"

namespace hb {
namespace {

__global__ __launch_bounds__(kFinThreads) void batch_alpha_kernel(const int32_t *__restrict__ plist,
                                                                 const BatchProb *__restrict__ probs)
{
    __shared__ double red[kFinThreads / 64];
    const BatchProb &P = probs[plist[blockIdx.x]];
    double alpha;
    alpha_step(P.part_ax, P.ax_tiles, P.st, red, true, &alpha);
}

__global__ __launch_bounds__(kFinThreads) void batch_beta_kernel(const int32_t *__restrict__ plist,
                                                                const BatchProb *__restrict__ probs)
{
    __shared__ double red[kFinThreads / 64];
    const BatchProb &P = probs[plist[blockIdx.x]];
    if (P.st->done | P.st->broke) return;
    beta_step(P.part_vec, P.vec_chunks, P.st, P.rho, P.hist, P.inv != nullptr, red, true);
}

// r -= alpha Ap on one chunk; the chunk's partial of r.r (Jacobi: of r.z, z =
// inv r, and of r.r in the second half of the partials).  FUSED: with the alpha step
// of the chunk's problem in every block.
template <bool FUSED>
__global__ __launch_bounds__(kVecThreads) void batch_residual_kernel(const WorkItem *__restrict__ items,
                                                                    const BatchProb *__restrict__ probs)
{
    __shared__ double red[kVecThreads / 64];
    const WorkItem it = items[blockIdx.x];
    const int32_t prob = uniform(it.prob), chunk = uniform(it.idx);
    const BatchProb &P = probs[prob];
    CgState *st = uniform(P.st);
    const int64_t n = uniform(P.NG);
    const auto r = to_global(uniform(P.r));
    const double *inv_p = uniform(P.inv);
    double rv[kVecEntries], av[kVecEntries], alpha, rr, rz;
    if (uniform(P.use32))
        load_chunk<false>(P.plan, n, chunk, threadIdx.x, r, to_global(uniform(P.Ap32)), to_global(uniform(P.halo32)), rv, av);
    else
        load_chunk<false>(P.plan, n, chunk, threadIdx.x, r, to_global(uniform(P.Ap)), to_global(uniform(P.halo)), rv, av);
    if constexpr (FUSED) {
        if (!alpha_step(uniform(P.part_ax), uniform(P.ax_tiles), st, red, chunk == 0, &alpha)) return;
    } else {
        if (st->done | st->broke) return;
        alpha = st->alpha;
    }
    store_chunk<false>(n, chunk, threadIdx.x, alpha, r, to_global(inv_p), inv_p != nullptr, rv, av, &rr, &rz);
    rr = block_sum(rr, red);
    if (inv_p) rz = block_sum(rz, red);
    if (threadIdx.x == 0) {
        const auto part = to_global(uniform(P.part_vec));
        part[chunk] = inv_p ? rz : rr;
        if (inv_p) part[uniform(P.vec_chunks) + chunk] = rr;
    }
}

// x += alpha p; p = r + beta p (Jacobi: p = inv r + beta p) on one chunk.  FUSED: with the beta step of the chunk's problem in every
// block.
template <bool FUSED>
__global__ __launch_bounds__(kVecThreads) void batch_update_kernel(const WorkItem *__restrict__ items,
                                                                  const BatchProb *__restrict__ probs)
{
    __shared__ double red[kVecThreads / 64];
    const WorkItem it = items[blockIdx.x];
    const int32_t prob = uniform(it.prob), chunk = uniform(it.idx);
    const BatchProb &P = probs[prob];
    CgState *st = uniform(P.st);
    if (st->done) return;
    if (st->broke) {
        if (chunk == 0 && threadIdx.x == 0) st->done = 1;
        return;
    }
    const double *inv_p = uniform(P.inv);
    const double alpha = st->alpha;
    double beta = st->beta;
    const int64_t NG = uniform(P.NG), lo = static_cast<int64_t>(chunk) * kVecChunk + threadIdx.x;
    const auto x = to_global(uniform(P.x));
    const auto p = to_global(uniform(P.p));
    const auto r = to_global(uniform(P.r));
    const auto inv = to_global(inv_p);
    double pv[kVecEntries], xv[kVecEntries], zv[kVecEntries];  // loaded ahead of the partials
#pragma unroll
    for (int k = 0; k < kVecEntries; ++k) {
        const int64_t i = lo + k * kVecThreads < NG ? lo + k * kVecThreads : NG - 1;
        pv[k] = p[i];
        xv[k] = x[i];
        zv[k] = r[i];
        if (inv_p) zv[k] *= inv[i];
    }
    if constexpr (FUSED)
        beta = beta_step(uniform(P.part_vec), uniform(P.vec_chunks), st, uniform(P.rho), uniform(P.hist),
                         inv_p != nullptr, red, chunk == 0);
#pragma unroll
    for (int k = 0; k < kVecEntries; ++k) {
        const int64_t i = lo + k * kVecThreads;
        if (i >= NG) continue;
        x[i] = xv[k] + alpha * pv[k];
        p[i] = zv[k] + beta * pv[k];
    }
}

}  // namespace

hb_status launch_batch_steps(const int32_t *plist, int np, const WorkItem *items, int nitems, const BatchProb *probs,
                             bool fused, hipStream_t s)
{
    if (np == 0 || nitems == 0) return HB_OK;
    if (fused) {
        batch_residual_kernel<true><<<nitems, kVecThreads, 0, s>>>(items, probs);
        batch_update_kernel<true><<<nitems, kVecThreads, 0, s>>>(items, probs);
    } else {
        batch_alpha_kernel<<<np, kFinThreads, 0, s>>>(plist, probs);
        batch_residual_kernel<false><<<nitems, kVecThreads, 0, s>>>(items, probs);
        batch_beta_kernel<<<np, kFinThreads, 0, s>>>(plist, probs);
        batch_update_kernel<false><<<nitems, kVecThreads, 0, s>>>(items, probs);
    }
    HB_HIP(hipGetLastError());
    return HB_OK;
}

}  // namespace hb
