// Batched CG in one persistent launch (Algorithm 1 for many independent
// problems; the latency model of the DOF Storage section, t = alpha + beta B,
// is why small problems want no per-step launches).
//
// The launch holds every running problem at once: problem p owns nwg_p
// workgroups, and those run its iterations back to back, each iteration three
// phases separated by a barrier among the problem's workgroups only:
//   operator  Ap = A p over the problem's tiles, partial of p.Ap
//   residual  alpha = rho_j / p.Ap from all partials (every workgroup sums
//             them in the same fixed order, so all hold the same alpha),
//             r -= alpha Ap (with the halo) over the workgroup's slice, partial of r.r (r.z)
//   update    beta = rho_{j+1} / rho_j likewise, x += alpha p,
//             p = r (or M^-1 r) + beta p over the slice.
// So no problem waits for another, and the host sees the device only between
// launches.  The stop tests, the history and the device state follow the
// single-block alpha and beta steps of the per-step runner exactly (cg_steps.h),
// so the host's handling of finished problems and of residual replacement is
// the same for both.
//
// Deadlock freedom: the launch is cooperative (the runtime guarantees that all
// its workgroups are resident at once, or refuses it), and a workgroup only
// waits for workgroups of its own problem.  Every wait is bounded: a barrier
// that spins past its limit raises *err and the launch ends.
//
// The kernel inlines the operator of each degree it is compiled for (one tile
// routine per degree and precision), so it runs at the occupancy of the most
// demanding of them (two workgroups to a compute unit); tiles use the 256-thread
// shape.  That suits the regime it is for, many small problems whose iterations
// are bound by the latency of dependent steps rather than by bandwidth; the host
// keeps large problems on the per-step launches.
//
// Bound by the barriers: each of the workgroups of an XCD writes its L2 back at each.
// So the host spreads the problems over one workgroup to a compute unit, not two
// (50 iterations: 32 problems of 4^3 N = 7 8.6 -> 4.7 ms, eight of N = 3 to 9 and
// 130000 to 2 million local nodes 10.8 -> 6.9, one of 24^3 N = 7 13.0 -> 10.6), a barrier
// releases and acquires once (10.1 -> 8.6, 13.3 -> 10.8, 15.1 -> 13.0), and a thread's
// entries of the vector steps are loaded four at a time.
#include <algorithm>
#include <cmath>
#include <mutex>
#include <type_traits>

#include "ax_impl.h"
#include "cg_steps.h"
#include "common.h"
#include "reduce.h"

namespace hb {
namespace {

// LDS of a tile of any degree in the launch
constexpr size_t kPersistLds =
    sizeof(double) * std::max({Shape<3, 0>::lds, Shape<5, 0>::lds, Shape<7, 0>::lds, Shape<9, 0>::lds});
constexpr uint32_t kSpinLimit = 1u << 22;  // polls of a barrier counter before giving up (~0.3 s)

// Arrive at barrier number `target / nwg` of one problem and wait for its other
// workgroups: the workgroup's writes, complete in every wave, are released (agent scope)
// before the arrival is counted, and the others' acquired after the count is complete.
// (A release writes the XCD's L2 back, for each workgroup on it; full fences on both
// sides did so twice.)  A problem's only workgroup (nwg 1) waits for itself alone.
// Returns false (every thread) if the wait timed out or another workgroup reported an
// error.
__device__ bool group_barrier(uint32_t *ctr, uint32_t target, int32_t nwg, int32_t *err, int *s_ok)
{
    __builtin_amdgcn_s_waitcnt(0);  // this wave's stores have reached the L2
    __syncthreads();
    if (nwg == 1) return true;
    if (threadIdx.x == 0) {
        int ok = 1;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        uint32_t spins = 0;
        while (__hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
            if (++spins > kSpinLimit || __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                __hip_atomic_fetch_or(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                ok = 0;
                break;
            }
            __builtin_amdgcn_s_sleep(2);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        *s_ok = ok;
    }
    __syncthreads();
    return *s_ok != 0;
}

// Ap = A p over tiles rank, rank + nwg, ... of the problem's walk (owned DOFs and
// halo); the workgroup's sum of the tiles' shares of p . A p.
template <int N, typename T, bool MASK>
__device__ __attribute__((always_inline)) inline double operator_share(unsigned char *lds, double *red, const BatchProb &P, const TilePlan &plan,
                                                                       int rank, int nwg)
{
    const AxFromBatch<T> from{to_const(&P)};
    const int tiles = plan.tiles();
    double dot = 0.0;
    for (int i = rank; i < tiles; i += nwg) {
        __syncthreads();  // the previous tile's LDS has been read
        dot += ax_tile<N, 0, T, true, MASK, kAssign>(reinterpret_cast<T *>(lds), red, from,
                                                   place_in_walk(plan, static_cast<uint32_t>(i)));
    }
    return dot;
}

template <bool MASK>
__device__ double operator_any(unsigned char *lds, double *red, const BatchProb &P, const PersistSlot &sl, int N, bool fp32, int rank, int nwg)
{
    switch (N) {
#define HB_PCASE(n)                                                                              \
    case n:                                                                                      \
        return fp32 ? operator_share<n, float, MASK>(lds, red, P, sl.plan, rank, nwg)            \
                    : operator_share<n, double, MASK>(lds, red, P, sl.plan, rank, nwg);
        HB_PCASE(3)
        HB_PCASE(5)
        HB_PCASE(7)
        HB_PCASE(9)
#undef HB_PCASE
    default: return 0.0;  // not reached: the host launches listed degrees only
    }
}

// A workgroup's share of a vector: entries first, first + stride, ... of a thread, `mine` of
// them (the same for all its threads; the last may lie past the end).  Four at a time, so
// that their loads are in flight together, then one at a time.
template <typename F>
__device__ __attribute__((always_inline)) inline void batches(int64_t first, int64_t stride, int mine, F &&f)
{
    int k = 0;
    for (; k + kVecEntries <= mine; k += kVecEntries) f(std::integral_constant<int, kVecEntries>{}, first + k * stride);
    for (; k < mine; ++k) f(std::integral_constant<int, 1>{}, first + k * stride);
}

// r -= alpha Ap (with the halo) on K of a thread's entries; adds to its sums of r.r and r.z.
template <int K, typename R, typename A, typename I>
__device__ __attribute__((always_inline)) inline void residual_entries(const TilePlan &plan, int64_t n, int64_t i0,
                                                                       int64_t stride, double alpha, R r, A Ap, A halo,
                                                                       I inv, double *rr, double *rz)
{
    using T = decltype(+Ap[0]);
    double rv[K], iv[K];
    T av[K];
    HaloNode<T> h[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int64_t i = i0 + k * stride < n ? i0 + k * stride : n - 1;
        rv[k] = r[i];
        av[k] = Ap[i];
        iv[k] = inv ? inv[i] : 0.0;
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int64_t i = i0 + k * stride < n ? i0 + k * stride : n - 1;
        const Node d = dof_node(plan, static_cast<uint32_t>(i));
        h[k].load(plan, halo, d.I, d.J, d.K);
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int64_t i = i0 + k * stride;
        if (i >= n) continue;
        const double v = rv[k] - alpha * (static_cast<double>(av[k]) + h[k].sum());
        r[i] = v;
        *rr += v * v;
        *rz += v * (iv[k] * v);
    }
}

template <bool MASK>
__global__ __launch_bounds__(kPersistThreads) void persist_kernel(const PersistWg *__restrict__ wgs,
                                                                 const PersistSlot *__restrict__ slots,
                                                                 const BatchProb *__restrict__ probs,
                                                                 uint32_t *__restrict__ bar, int32_t *__restrict__ err)
{
    __shared__ double red[kPersistThreads / 64];
    __shared__ int s_ok;
    __shared__ __attribute__((aligned(16))) unsigned char lds[kPersistLds];
    const int t = threadIdx.x;
    const int32_t prob = uniform(wgs[blockIdx.x].prob), rank = uniform(wgs[blockIdx.x].rank);
    const PersistSlot &sl = slots[prob];
    const int32_t nwg = uniform(sl.nwg), budget = uniform(sl.iters);
    const BatchProb &P = probs[prob];
    CgState *st = uniform(P.st);
    const int N = uniform(P.N);
    const bool fp32 = uniform(P.use32) != 0;
    const int64_t n = uniform(P.NG);
    double *rho = uniform(P.rho), *hist = uniform(P.hist);
    double *part_ax = uniform(P.part_ax), *part_vec = uniform(P.part_vec);
    const auto x = to_global(uniform(P.x)), r = to_global(uniform(P.r)), p = to_global(uniform(P.p));
    const auto Ap = to_global(uniform(P.Ap));
    const auto Ap32 = to_global(uniform(P.Ap32));
    const auto halo = to_global(uniform(P.halo));
    const auto halo32 = to_global(uniform(P.halo32));
    const auto inv = to_global(uniform(P.inv));
    uint32_t *ctr = bar + prob;
    uint32_t passed = 0;

    // the starting state, read by every workgroup before any of them changes it
    int32_t it = uniform(st->it), iters = uniform(st->iters), done = uniform(st->done);
    int32_t pending = uniform(st->pending), status = uniform(st->status);
    const int32_t max_iter = uniform(st->max_iter);
    const double stop_res = uniform(st->stop_res), rtol = uniform(st->rtol);
    double alpha = uniform(st->alpha), beta = uniform(st->beta), pAp = uniform(st->pAp);
    double rho_j = uniform(st->rho);
    if (!group_barrier(ctr, ++passed * nwg, nwg, err, &s_ok)) return;

    const int64_t first = static_cast<int64_t>(rank) * kPersistThreads + t;
    const int64_t stride = static_cast<int64_t>(nwg) * kPersistThreads;
    const int64_t left = n - static_cast<int64_t>(rank) * kPersistThreads;
    const int mine = left > 0 ? static_cast<int>((left + stride - 1) / stride) : 0;
    for (int k = 0; k < budget; ++k) {
        // alpha step: a stop decided by the last beta step takes effect here
        if (done) break;
        if (pending) {
            done = 1;
            break;
        }
        const double d = operator_any<MASK>(lds, red, P, sl, N, fp32, rank, nwg);
        if (t == 0) part_ax[rank] = d;
        if (!group_barrier(ctr, ++passed * nwg, nwg, err, &s_ok)) return;
        pAp = uniform(sum_partials(part_ax, nwg, red));
        const int j = it + 1;
        it = j;
        if (!(pAp > 0.0) || !isfinite(pAp)) {
            done = 1;
            status = HB_ERR_BREAKDOWN;
            break;
        }
        alpha = uniform(rho_j / pAp);

        // residual step
        double rr = 0.0, rz = 0.0;
        batches(first, stride, mine, [&](auto KK, int64_t i0) {
            if (fp32)
                residual_entries<decltype(KK)::value>(sl.plan, n, i0, stride, alpha, r, Ap32, halo32, inv, &rr, &rz);
            else
                residual_entries<decltype(KK)::value>(sl.plan, n, i0, stride, alpha, r, Ap, halo, inv, &rr, &rz);
        });
        rr = block_sum(rr, red);
        if (inv) rz = block_sum(rz, red);
        if (t == 0) {
            part_vec[rank] = inv ? rz : rr;
            if (inv) part_vec[nwg + rank] = rr;
        }
        if (!group_barrier(ctr, ++passed * nwg, nwg, err, &s_ok)) return;
        const double rho_new = uniform(sum_partials(part_vec, nwg, red));
        const double rrs = inv ? uniform(sum_partials(part_vec + nwg, nwg, red)) : rho_new;

        // beta step (as beta_step): history, stop tests; the update below still runs
        beta = uniform(rho_new / rho_j);
        if (rank == 0 && t == 0) {
            rho[j + 1] = rho_new;
            hist[j + 1] = sqrt(rrs);
        }
        iters = j + 1;
        if (!isfinite(rho_new) || !isfinite(rrs)) {
            pending = 1;
            status = HB_ERR_BREAKDOWN;
        } else if (rho_new == 0.0 || sqrt(rrs) <= stop_res) {
            pending = 1;
            status = HB_OK;
        } else if (j + 1 >= max_iter) {
            pending = 1;
            status = rtol >= 0.0 ? HB_ERR_NOT_CONVERGED : HB_OK;
        }
        rho_j = rho_new;

        // update step
        batches(first, stride, mine, [&](auto KK, int64_t i0) {
            constexpr int K = decltype(KK)::value;
            double pv[K], xv[K], zv[K];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int64_t i = i0 + k * stride < n ? i0 + k * stride : n - 1;
                pv[k] = p[i];
                xv[k] = x[i];
                zv[k] = r[i];
                if (inv) zv[k] *= inv[i];
            }
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int64_t i = i0 + k * stride;
                if (i >= n) continue;
                x[i] = xv[k] + alpha * pv[k];
                p[i] = zv[k] + beta * pv[k];
            }
        });
        if (!group_barrier(ctr, ++passed * nwg, nwg, err, &s_ok)) return;
    }
    if (rank == 0 && t == 0) {
        st->it = it;
        st->iters = iters;
        st->alpha = alpha;
        st->beta = beta;
        st->pAp = pAp;
        st->rho = rho_j;
        st->done = done;
        st->pending = pending;
        st->status = status;
    }
}

std::once_flag g_cap_once;
int g_cap = 0, g_cus = 0;

}  // namespace

bool persist_degree(int N) { return N == 3 || N == 5 || N == 7 || N == 9; }

int persist_capacity()
{
    std::call_once(g_cap_once, [] {
        int dev = 0, cus = 0, coop = 0, per_cu = 0, per_cu_d = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess || !coop ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, persist_kernel<false>, kPersistThreads, 0) !=
                hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu_d, persist_kernel<true>, kPersistThreads, 0) !=
                hipSuccess) {
            (void)hipGetLastError();
            g_cap = 0;
            return;
        }
        g_cap = cus * std::min(per_cu, per_cu_d);
        g_cus = cus;
    });
    return g_cap;
}

int persist_spread()
{
    (void)persist_capacity();
    return g_cus;
}

hb_status launch_batch_persistent(bool dirichlet, const PersistWg *wgs, int nwg, const PersistSlot *slots,
                                  const BatchProb *probs, uint32_t *bar, int32_t *err, hipStream_t s)
{
    static_assert(Shape<3, 0>::threads == kPersistThreads && Shape<5, 0>::threads == kPersistThreads &&
                      Shape<7, 0>::threads == kPersistThreads && Shape<9, 0>::threads == kPersistThreads,
                  "every degree of the persistent kernel tiles with its workgroup size");
    if (nwg == 0) return HB_OK;
    if (nwg > persist_capacity())
        return fail(HB_ERR_INVALID_ARG, "persistent batch: more workgroups than the device holds at once");
    void *args[] = {&wgs, &slots, &probs, &bar, &err};
    const void *fn = dirichlet ? reinterpret_cast<const void *>(&persist_kernel<true>)
                               : reinterpret_cast<const void *>(&persist_kernel<false>);
    HB_HIP(hipLaunchCooperativeKernel(fn, dim3(nwg), dim3(kPersistThreads), args, 0, s));
    return HB_OK;
}

}  // namespace hb
