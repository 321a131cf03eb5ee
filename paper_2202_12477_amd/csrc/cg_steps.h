// The two single-block scalar steps of a CG iteration (Algorithm 1), shared
// by the one-problem kernels and the batched kernels (one block per problem).
#pragma once

#include <cmath>

#include "common.h"
#include "reduce.h"

namespace hb {

constexpr int kFinThreads = 1024;
constexpr int kVecThreads = 256;

// Fixed-order sum of partial[0..n) by one block (call from every thread).
// The partials were written by an earlier kernel on the stream.
__device__ inline double sum_partials(const double *partial, int n, double *scratch)
{
    // eight loads in flight per thread, added in index order (the same sums as a
    // plain strided loop, without waiting on each load; past the end a thread
    // adds zeros, which leaves its sum unchanged)
    double s = 0.0;
    const int step = blockDim.x;
    for (int i = threadIdx.x; i < n; i += 8 * step) {
        double v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = i + k * step < n ? partial[i + k * step] : 0.0;
#pragma unroll
        for (int k = 0; k < 8; ++k) s += v[k];
    }
    return block_sum(s, scratch);
}

// The alpha step, iteration j = it + 1 (= iters): alpha = rho_j / p.Ap, or stop on
// breakdown (p.Ap <= 0 or not finite), or apply a stop decided by the previous
// beta.  Returns whether the iteration goes on, and its alpha, in every thread;
// `writer` (one block) records them in the state.  Every block of a launch may
// call it: the fields it reads are not written in the same launch, except done
// where pending is set, and either makes every block return.
__device__ inline bool alpha_step(const double *__restrict__ partial, int nblk, CgState *st, double *scratch,
                                  bool writer, double *alpha)
{
    const bool lead = writer && threadIdx.x == 0;
    if (st->done) return false;
    if (st->pending) {
        if (lead) st->done = 1;
        return false;
    }
    const int j = st->iters;
    const double rho_j = st->rho;
    const double pAp = sum_partials(partial, nblk, scratch);
    const bool ok = pAp > 0.0 && isfinite(pAp);
    *alpha = rho_j / pAp;
    if (lead) {
        st->it = j;
        st->rho_j = rho_j;
        st->pAp = pAp;
        if (ok) {
            st->alpha = *alpha;
        } else {
            st->broke = 1;
            st->status = HB_ERR_BREAKDOWN;
        }
    }
    return ok;
}

// What the beta step of iteration j leaves in the state and the histories.
__device__ inline void record_beta(CgState *st, int j, double beta, double rho_new, double rr,
                                   double *__restrict__ rho, double *__restrict__ hist)
{
    st->beta = beta;
    st->rho = rho_new;
    rho[j + 1] = rho_new;
    hist[j + 1] = sqrt(rr);
    st->iters = j + 1;
    // this iteration's update still runs; the next alpha turns pending into done
    if (!isfinite(rho_new) || !isfinite(rr)) {
        st->pending = 1;
        st->status = HB_ERR_BREAKDOWN;
    } else if (rho_new == 0.0 || sqrt(rr) <= st->stop_res) {
        st->pending = 1;
        st->status = HB_OK;
    } else if (j + 1 >= st->max_iter) {
        st->pending = 1;
        st->status = st->rtol >= 0.0 ? HB_ERR_NOT_CONVERGED : HB_OK;
    }
}

// The beta step: rho_{j+1} = r.r, beta, history, convergence / iteration-cap test.
// With the Jacobi preconditioner (pc) the partials hold r.z and then r.r: rho and
// beta use r.z, the history and the stop test ||r||.  Returns beta in every
// thread; `writer` records it (the fields it writes are not read in the same
// launch).  Not called once the solve is done.
__device__ inline double beta_step(const double *__restrict__ partial, int nblk, CgState *st,
                                   double *__restrict__ rho, double *__restrict__ hist, bool pc, double *scratch,
                                   bool writer)
{
    const int j = st->it;
    const double rho_j = st->rho_j;
    const double rho_new = sum_partials(partial, nblk, scratch);
    const double rr = pc ? sum_partials(partial + nblk, nblk, scratch) : rho_new;
    const double beta = rho_new / rho_j;
    if (writer && threadIdx.x == 0) record_beta(st, j, beta, rho_new, rr, rho, hist);
    return beta;
}

// The entries of one chunk of r and Ap that a thread works on: kVecChunk / kVecThreads
// of them, all in flight, Ap with the halo added.  Loaded before alpha is known, so
// that in the fused form these loads and the partials' overlap.  t: the thread's
// number among the chunk's kVecThreads.  (With 32-bit entry numbers, 76 registers: six
// waves to a SIMD; with 64-bit ones 84 and five, 16 boxes with Jacobi 1.5% slower, 50^3
// 95.9 against 94.5 ms per 100 iterations.)
constexpr int kVecEntries = kVecChunk / kVecThreads;
template <bool NT, typename R, typename A, typename H>
__device__ __attribute__((always_inline)) inline void load_chunk(const TilePlan &plan, int64_t n, int chunk, int t, R r, A Ap,
                                                                 H halo, double (&rv)[kVecEntries],
                                                                 double (&av)[kVecEntries])
{
    using T = decltype(+Ap[0]);
    const uint32_t lo = static_cast<uint32_t>(chunk) * kVecChunk + t, last = static_cast<uint32_t>(n) - 1;
    T a[kVecEntries];  // converted once every load is on its way
#pragma unroll
    for (int k = 0; k < kVecEntries; ++k) {
        const uint32_t i = min(lo + k * kVecThreads, last);
        rv[k] = NT ? __builtin_nontemporal_load(&r[i]) : r[i];
        a[k] = NT ? __builtin_nontemporal_load(&Ap[i]) : Ap[i];
    }
    HaloNode<T> h[kVecEntries];
#pragma unroll
    for (int k = 0; k < kVecEntries; ++k) {
        const Node d = dof_node(plan, min(lo + k * kVecThreads, last));
        h[k].load(plan, halo, d.I, d.J, d.K);
    }
#pragma unroll
    for (int k = 0; k < kVecEntries; ++k) av[k] = static_cast<double>(a[k]) + h[k].sum();
}
// r <- rv - alpha av on the chunk; this thread's sums of r.r and (pc) r.z, z = inv r.
template <bool NT, typename R, typename I>
__device__ __attribute__((always_inline)) inline void store_chunk(int64_t n, int chunk, int t, double alpha, R r, I inv,
                                                                  bool pc, const double (&rv)[kVecEntries],
                                                                  const double (&av)[kVecEntries], double *rr,
                                                                  double *rz)
{
    const int64_t lo = static_cast<int64_t>(chunk) * kVecChunk + t;
    *rr = *rz = 0.0;
#pragma unroll
    for (int k = 0; k < kVecEntries; ++k) {
        const int64_t i = lo + k * kVecThreads;
        if (i >= n) continue;
        const double v = rv[k] - alpha * av[k];
        if (NT)
            __builtin_nontemporal_store(v, &r[i]);
        else
            r[i] = v;
        *rr += v * v;
        if (pc) *rz += v * (inv[i] * v);
    }
}

}  // namespace hb
