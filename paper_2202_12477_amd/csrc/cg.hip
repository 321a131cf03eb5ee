// Kernels of the conjugate-gradient iteration (Algorithm 1; fused as in the
// Conjugate gradient Iteration section, with every scalar kept on the device so
// the host never waits inside an iteration).
//
// An iteration is these steps on one stream, identical for every iteration (the
// iteration number lives in the device state): five launches, or three where the
// partials are few and each block of the residual and update steps sums them itself,
// or two on very short vectors (tail_kernel):
//   operator  Ap = A p, block partials of p.Ap              (ax*.hip)
//   alpha     one block: p.Ap from the partials, alpha = rho_j / p.Ap
//   residual  r -= alpha Ap (the tiles' halo added as Ap is read), block partials of r.r
//   beta      one block: rho_{j+1} = r.r, beta = rho_{j+1} / rho_j, history, stop test
//   update    x += alpha p; p = r + beta p
// Streaming kernels never wait for each other's blocks and issue no
// device-scope fences: the single-block kernels finish the reductions in a
// fixed order after the kernel boundary has made the partials visible.
#include <climits>
#include <cmath>
#include <type_traits>

#include "cg_steps.h"
#include "common.h"
#include "reduce.h"

namespace hb {
namespace {

template <typename V>
__global__ __launch_bounds__(kVecThreads) void zero_kernel(V *__restrict__ v, int64_t n)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        v[i] = V(0);
}

__global__ void setup_state_kernel(CgState *st, int max_iter, double rtol)
{
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    st->bb = st->alpha = st->beta = st->pAp = st->rho = st->rho_j = 0.0;
    st->rtol = rtol;
    st->stop_res = -1.0;
    st->max_iter = max_iter;
    st->it = -1;
    st->iters = 0;
    st->done = 0;
    st->pending = 0;
    st->broke = 0;
    st->status = HB_OK;
}

// r0 = b - A x0 (Ap holds A x0 unless x0 = 0), p = r0; partials of r0.r0 and b.b.
// PC (Jacobi): p = z0 = inv r0, and a third partial array of r0.z0.
template <typename TAp, bool PC>
__global__ __launch_bounds__(kVecThreads) void init_kernel(int64_t n, const double *__restrict__ b,
                                                          double *__restrict__ x, double *__restrict__ r,
                                                          double *__restrict__ p, const TAp *__restrict__ Ap,
                                                          int x0_zero, const double *__restrict__ inv,
                                                          double *__restrict__ partial)
{
    __shared__ double red[kVecThreads / 64];
    double rr = 0.0, bb = 0.0, rz = 0.0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const double bi = b[i];
        const double ri = x0_zero ? bi : bi - static_cast<double>(Ap[i]);
        r[i] = ri;
        if constexpr (PC) {
            const double zi = inv[i] * ri;
            p[i] = zi;
            rz += ri * zi;
        } else {
            p[i] = ri;
        }
        if (x0_zero) x[i] = 0.0;
        rr += ri * ri;
        bb += bi * bi;
    }
    rr = block_sum(rr, red);
    bb = block_sum(bb, red);
    if constexpr (PC) rz = block_sum(rz, red);
    if (threadIdx.x == 0) {
        partial[blockIdx.x] = rr;
        partial[gridDim.x + blockIdx.x] = bb;
        if constexpr (PC) partial[2 * gridDim.x + blockIdx.x] = rz;
    }
}

__global__ __launch_bounds__(kFinThreads) void init_finish_kernel(const double *__restrict__ partial, int nblk,
                                                                 int pc, CgState *st, double *__restrict__ rho,
                                                                 double *__restrict__ hist)
{
    __shared__ double red[kFinThreads / 64];
    const double rho0 = sum_partials(partial, nblk, red);  // r0.r0: the stop tests
    const double bb = sum_partials(partial + nblk, nblk, red);
    const double rz0 = pc ? sum_partials(partial + 2 * nblk, nblk, red) : rho0;
    if (threadIdx.x != 0) return;
    st->bb = bb;
    st->rho = rz0;
    rho[0] = rz0;
    hist[0] = sqrt(rho0);
    st->stop_res = st->rtol >= 0.0 ? st->rtol * sqrt(bb) : -1.0;
    if (!isfinite(rho0)) {
        st->done = 1;
        st->status = HB_ERR_NONFINITE;
    } else if (rho0 == 0.0 || sqrt(rho0) <= st->stop_res) {
        st->done = 1;  // already solved
    } else if (st->max_iter == 0) {
        st->done = 1;
        st->status = st->rtol >= 0.0 ? HB_ERR_NOT_CONVERGED : HB_OK;
    }
}

__global__ __launch_bounds__(kFinThreads) void alpha_kernel(const double *__restrict__ partial, int nblk, CgState *st)
{
    __shared__ double red[kFinThreads / 64];
    double alpha;
    alpha_step(partial, nblk, st, red, true, &alpha);
}

__device__ inline void store_partials(bool pc, double rr, double rz, double *__restrict__ partial, double *red)
{
    rr = block_sum(rr, red);
    if (pc) rz = block_sum(rz, red);
    if (threadIdx.x == 0) {
        partial[blockIdx.x] = pc ? rz : rr;
        if (pc) partial[gridDim.x + blockIdx.x] = rr;
    }
}

// r -= alpha Ap, the halo added to Ap on the way; partials of r.r (PC: of r.z, z =
// inv r, then of r.r).  One chunk to a block.  NT: r and Ap non-temporally.  FUSED:
// with the alpha step in every block.
// Bound by HBM: 24 N_G bytes and the halo (0.33 N_G entries at N = 7).  32^3 N = 7:
// 50 us; 57 us with each entry's halo loads waited for in turn (HaloNode now has a
// thread's four entries in flight), 84 us by DOF rows with the row's place worked out
// once, 39 us without a halo -- but adding it in a launch of its own, with the alpha
// step beside it, took 27 us.
template <typename TAp, bool PC, bool NT, bool FUSED>
__global__ __launch_bounds__(kVecThreads) void residual_kernel(TilePlan plan, int64_t n, double *__restrict__ r,
                                                              const TAp *__restrict__ Ap,
                                                              const TAp *__restrict__ halo,
                                                              const double *__restrict__ inv,
                                                              const double *__restrict__ part_ax, int nax,
                                                              double *__restrict__ partial, CgState *st)
{
    __shared__ double red[kVecThreads / 64];
    double rv[kVecEntries], av[kVecEntries], alpha, rr, rz;
    load_chunk<NT>(plan, n, blockIdx.x, threadIdx.x, r, Ap, halo, rv, av);
    if constexpr (FUSED) {
        if (!alpha_step(part_ax, nax, st, red, blockIdx.x == 0, &alpha)) return;
    } else {
        if (st->done | st->broke) return;
        alpha = st->alpha;
    }
    store_chunk<NT>(n, blockIdx.x, threadIdx.x, alpha, r, inv, PC, rv, av, &rr, &rz);
    store_partials(PC, rr, rz, partial, red);
}

__global__ __launch_bounds__(kFinThreads) void beta_kernel(const double *__restrict__ partial, int nblk, int pc,
                                                          CgState *st, double *__restrict__ rho,
                                                          double *__restrict__ hist)
{
    __shared__ double red[kFinThreads / 64];
    if (st->done | st->broke) return;
    beta_step(partial, nblk, st, rho, hist, pc != 0, red, true);
}

// x += alpha p; p = r + beta p (PC: p = inv r + beta p).  FUSED: with the beta step
// in every block.  NT: x and r non-temporally (not read again before the next update
// or residual step, where the vectors do not stay in the caches until then); p
// with plain stores, which the operator gathers next.
// One chunk to a block as in the residual step, which leaves r in the same L2, and all
// of a thread's loads at once.  Bound by HBM: 40 N_G bytes.  With the residual step
// before it, against two entries to a thread one after the other, in half as large
// blocks: 50^3 N = 7 489 -> 468 us, 32^3 125 -> 123 us, 11x10x9 N = 11 (fused, FP32
// operator) 23.5 -> 20.5 us (18.5 with the residual step's FP32 halo as it is now).
template <bool PC, bool NT, bool FUSED>
__global__ __launch_bounds__(kVecThreads) void update_kernel(int64_t n, double *__restrict__ x, double *__restrict__ p,
                                                            const double *__restrict__ r,
                                                            const double *__restrict__ inv,
                                                            const double *__restrict__ part, int npart, CgState *st,
                                                            double *__restrict__ rho, double *__restrict__ hist)
{
    __shared__ double red[kVecThreads / 64];
    if (st->done) return;
    if (st->broke) {
        if (blockIdx.x == 0 && threadIdx.x == 0) st->done = 1;
        return;
    }
    const double alpha = st->alpha;
    double beta = st->beta;
    const int64_t lo = static_cast<int64_t>(blockIdx.x) * kVecChunk + threadIdx.x;
    double pv[kVecEntries], xv[kVecEntries], zv[kVecEntries];  // ahead of the partials
#pragma unroll
    for (int k = 0; k < kVecEntries; ++k) {
        const int64_t i = lo + k * kVecThreads < n ? lo + k * kVecThreads : n - 1;
        pv[k] = p[i];
        xv[k] = NT ? __builtin_nontemporal_load(&x[i]) : x[i];
        zv[k] = NT ? __builtin_nontemporal_load(&r[i]) : r[i];
        if constexpr (PC) zv[k] *= inv[i];
    }
    if constexpr (FUSED) beta = beta_step(part, npart, st, rho, hist, PC, red, blockIdx.x == 0);
#pragma unroll
    for (int k = 0; k < kVecEntries; ++k) {
        const int64_t i = lo + k * kVecThreads;
        if (i >= n) continue;
        const double xn = xv[k] + alpha * pv[k];
        if (NT)
            __builtin_nontemporal_store(xn, &x[i]);
        else
            x[i] = xn;
        p[i] = zv[k] + beta * pv[k];
    }
}

// The four steps after the operator -- alpha, r -= alpha Ap with r.r, beta,
// x += alpha p; p = r + beta p (inv: p = inv r + beta p) -- in one workgroup, for
// vectors so short that one workgroup streams them in less time than more launches
// take.  Every load is issued at the start (none depends on another), so the kernel
// takes one trip to memory.  Chunks and orders of summation are those of the
// launches, so the results are the same bits.
template <typename TAp>
__global__ __launch_bounds__(kFinThreads) void tail_kernel(TilePlan plan, int64_t n, double *__restrict__ x,
                                                          double *__restrict__ p, double *__restrict__ r,
                                                          const TAp *__restrict__ Ap, const TAp *__restrict__ halo,
                                                          const double *__restrict__ inv,
                                                          const double *__restrict__ part_ax, int nax, CgState *st,
                                                          double *__restrict__ rho, double *__restrict__ hist)
{
    static_assert(kCgTailMax == kVecChunk * (kFinThreads / kVecThreads), "a chunk to each group of kVecThreads threads");
    constexpr int groups = kFinThreads / kVecThreads, waves = kVecThreads / 64;
    __shared__ double red[kFinThreads / 64], vred[2][groups * waves];
    const int chunk = threadIdx.x / kVecThreads, t = threadIdx.x % kVecThreads;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double rv[kVecEntries] = {}, av[kVecEntries] = {}, pv[kVecEntries], xv[kVecEntries], iv[kVecEntries], alpha;
    const int64_t lo = static_cast<int64_t>(chunk) * kVecChunk + t;
    // (an empty chunk's waves stay out of the others' way: 8^3 N = 1, one chunk, 11.5 us an
    // iteration against 12.8 when they loaded a valid entry's values)
    if (static_cast<int64_t>(chunk) * kVecChunk < n) {
        load_chunk<false>(plan, n, chunk, t, r, Ap, halo, rv, av);
#pragma unroll
        for (int k = 0; k < kVecEntries; ++k) {
            const int64_t i = lo + k * kVecThreads < n ? lo + k * kVecThreads : n - 1;
            pv[k] = p[i];
            xv[k] = x[i];
            iv[k] = inv ? inv[i] : 1.0;
        }
    }
    if (!alpha_step(part_ax, nax, st, red, true, &alpha)) {
        __syncthreads();
        if (threadIdx.x == 0 && st->broke) st->done = 1;
        return;
    }
    double rr = 0.0, rz = 0.0;
#pragma unroll
    for (int k = 0; k < kVecEntries; ++k) {
        rv[k] -= alpha * av[k];
        if (lo + k * kVecThreads >= n) continue;
        rr += rv[k] * rv[k];
        if (inv) rz += rv[k] * (iv[k] * rv[k]);
    }
    rr = wave_sum(rr);
    rz = wave_sum(rz);
    if (lane == 0) {
        vred[0][wave] = rr;
        vred[1][wave] = rz;
    }
    __syncthreads();
    // the chunks' partials, then their sum as sum_partials has it
    double pr = 0.0, pz = 0.0;
    if (lane < groups && static_cast<int64_t>(lane) * kVecChunk < n) {
        for (int i = 0; i < waves; ++i) pr += vred[0][lane * waves + i];
        for (int i = 0; i < waves; ++i) pz += vred[1][lane * waves + i];
    }
    rr = wave_sum(pr);
    const double rho_new = inv ? wave_sum(pz) : rr;
    const int j = st->iters;
    const double beta = rho_new / st->rho;
    __syncthreads();  // every thread has read the state
    if (threadIdx.x == 0) record_beta(st, j, beta, rho_new, rr, rho, hist);
#pragma unroll
    for (int k = 0; k < kVecEntries; ++k) {
        const int64_t i = lo + k * kVecThreads;
        if (i >= n) continue;
        r[i] = rv[k];
        x[i] = xv[k] + alpha * pv[k];
        p[i] = (inv ? iv[k] * rv[k] : rv[k]) + beta * pv[k];
    }
}

// r = b - t; partials of r.r (and, with inv, of r.z, z = inv r, after them).
__global__ __launch_bounds__(kVecThreads) void residual_norm_kernel(int64_t n, const double *__restrict__ b,
                                                                   const double *__restrict__ t,
                                                                   double *__restrict__ r,
                                                                   const double *__restrict__ inv,
                                                                   double *__restrict__ partial)
{
    __shared__ double red[kVecThreads / 64];
    double rr = 0.0, rz = 0.0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const double ri = b[i] - t[i];
        r[i] = ri;
        rr += ri * ri;
        if (inv) rz += ri * (inv[i] * ri);
    }
    rr = block_sum(rr, red);
    if (threadIdx.x == 0) partial[blockIdx.x] = rr;
    if (inv) {
        rz = block_sum(rz, red);
        if (threadIdx.x == 0) partial[gridDim.x + blockIdx.x] = rz;
    }
}

// rho_iters = r.r (Jacobi, pc: r.z), history entry iters = ||r||, *out = r.r.
__global__ __launch_bounds__(kFinThreads) void replace_finish_kernel(const double *__restrict__ partial, int nblk,
                                                                    int pc, CgState *st, double *__restrict__ rho,
                                                                    double *__restrict__ hist,
                                                                    double *__restrict__ out)
{
    __shared__ double red[kFinThreads / 64];
    const double rr = sum_partials(partial, nblk, red);
    const double rz = pc ? sum_partials(partial + nblk, nblk, red) : rr;
    if (threadIdx.x != 0) return;
    const int j = st->iters;
    st->rho = rz;
    rho[j] = rz;
    hist[j] = sqrt(rr);
    *out = rr;
}

// Continue after a residual replacement: the next alpha starts iteration `iters`.
__global__ void resume_kernel(CgState *st, double stop_res)
{
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    st->stop_res = stop_res;
    st->it = st->iters - 1;
    st->done = 0;
    st->pending = 0;
    st->broke = 0;
    st->status = HB_OK;
}

__global__ __launch_bounds__(kFinThreads) void sum_kernel(const double *__restrict__ partial, int nblk,
                                                         double *__restrict__ out)
{
    __shared__ double red[kFinThreads / 64];
    const double s = sum_partials(partial, nblk, red);
    if (threadIdx.x == 0) *out = s;
}

__global__ __launch_bounds__(kVecThreads) void axpy_kernel(int64_t n, double *__restrict__ x,
                                                          const double *__restrict__ d)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        x[i] += d[i];
}

}  // namespace

// Two entries per thread, up to 32768 workgroups: with 2048 workgroups (four or
// more entries each) a CG iteration at 32^3 N=7 took 378 us against 357 us, and
// the streaming kernels need many loads in flight (see also zero_blocks).
int vec_blocks(int64_t n)
{
    const int64_t want = (n + kVecThreads * 2 - 1) / (kVecThreads * 2);
    return static_cast<int>(want < 1 ? 1 : (want > 32768 ? 32768 : want));
}

// Clearing takes one entry per thread and up to 32768 workgroups: a store-only
// kernel needs many more stores in flight than the vector kernels' 2048-workgroup
// grid gives (the 32^3 N=7 vector: 15.7 us against 18.4 us with 2048 workgroups).
inline int zero_blocks(int64_t n)
{
    const int64_t want = (n + kVecThreads - 1) / kVecThreads;
    return static_cast<int>(want < 1 ? 1 : (want > 32768 ? 32768 : want));
}

template <typename V>
hb_status zero_any(V *v, int64_t n, hipStream_t s)
{
    if (n == 0) return HB_OK;
    zero_kernel<V><<<zero_blocks(n), kVecThreads, 0, s>>>(v, n);
    HB_HIP(hipGetLastError());
    return HB_OK;
}

hb_status launch_zero(double *v, int64_t n, hipStream_t s) { return zero_any(v, n, s); }
hb_status launch_zero(float *v, int64_t n, hipStream_t s) { return zero_any(v, n, s); }

hb_status launch_cg_setup_state(CgState *st, int max_iter, double rtol, hipStream_t s)
{
    setup_state_kernel<<<1, 64, 0, s>>>(st, max_iter, rtol);
    HB_HIP(hipGetLastError());
    return HB_OK;
}

template <typename TAp>
hb_status launch_cg_init(int64_t n, const double *b, double *x, double *r, double *p, TAp *Ap, int x0_zero,
                         CgWork &w, CgState *st, hipStream_t s)
{
    const int g = vec_blocks(n);
    if (w.pc)
        init_kernel<TAp, true><<<g, kVecThreads, 0, s>>>(n, b, x, r, p, Ap, x0_zero, w.jinv, w.part_vec);
    else
        init_kernel<TAp, false><<<g, kVecThreads, 0, s>>>(n, b, x, r, p, Ap, x0_zero, nullptr, w.part_vec);
    init_finish_kernel<<<1, kFinThreads, 0, s>>>(w.part_vec, g, w.pc ? 1 : 0, st, w.rho, w.hist);
    HB_HIP(hipGetLastError());
    return HB_OK;
}

template <typename TAp>
hb_status launch_cg_steps(int64_t n, double *x, double *p, double *r, const TAp *Ap, const TilePlan &plan,
                          const TAp *halo, const double *inv, CgWork &w, CgState *st, hipStream_t s)
{
    const int nax = plan.tiles(), nvec = vec_chunks(n);
    const bool fused = nax <= kFuseMax && nvec <= kFuseMax;
    // r, p and Ap streamed together leave the caches; x too (32^3 N = 7, 273 MB in
    // the three: 118 us for the vector steps with x alone non-temporal, 121 us with
    // r and Ap as well, 126 us with neither; 50^3, 1020 MB: 598, 548 and 615 us; 3M
    // DOFs: 37, 38 and 35 us)
    const uint64_t bytes = static_cast<uint64_t>(n) * 8;
    const bool nt_r = 3 * bytes > (uint64_t(512) << 20), nt_x = 4 * bytes > (uint64_t(256) << 20);
    auto pick = [](bool v, auto &&f) { return v ? f(std::true_type{}) : f(std::false_type{}); };
    if (!fused) alpha_kernel<<<1, kFinThreads, 0, s>>>(w.part_ax, nax, st);
    pick(inv != nullptr, [&](auto PC) {
        pick(nt_r, [&](auto NT) {
            pick(fused, [&](auto F) {
                residual_kernel<TAp, PC.value, NT.value, F.value><<<nvec, kVecThreads, 0, s>>>(
                    plan, n, r, Ap, halo, inv, w.part_ax, nax, w.part_vec, st);
            });
        });
        if (!fused) beta_kernel<<<1, kFinThreads, 0, s>>>(w.part_vec, nvec, inv ? 1 : 0, st, w.rho, w.hist);
        pick(nt_x, [&](auto NT) {
            pick(fused, [&](auto F) {
                update_kernel<PC.value, NT.value, F.value><<<nvec, kVecThreads, 0, s>>>(n, x, p, r, inv, w.part_vec, nvec,
                                                                                     st, w.rho, w.hist);
            });
        });
    });
    HB_HIP(hipGetLastError());
    return HB_OK;
}

template <typename TAp>
hb_status launch_cg_tail(int64_t n, double *x, double *p, double *r, const TAp *Ap, const TilePlan &plan,
                         const TAp *halo, const double *inv, CgWork &w, CgState *st, hipStream_t s)
{
    tail_kernel<TAp><<<1, kFinThreads, 0, s>>>(plan, n, x, p, r, Ap, halo, inv, w.part_ax, plan.tiles(), st, w.rho,
                                               w.hist);
    HB_HIP(hipGetLastError());
    return HB_OK;
}

template hb_status launch_cg_init<double>(int64_t, const double *, double *, double *, double *, double *, int,
                                          CgWork &, CgState *, hipStream_t);
template hb_status launch_cg_init<float>(int64_t, const double *, double *, double *, double *, float *, int,
                                         CgWork &, CgState *, hipStream_t);
template hb_status launch_cg_tail<double>(int64_t, double *, double *, double *, const double *, const TilePlan &,
                                          const double *, const double *, CgWork &, CgState *, hipStream_t);
template hb_status launch_cg_tail<float>(int64_t, double *, double *, double *, const float *, const TilePlan &,
                                         const float *, const double *, CgWork &, CgState *, hipStream_t);
template hb_status launch_cg_steps<double>(int64_t, double *, double *, double *, const double *, const TilePlan &,
                                           const double *, const double *, CgWork &, CgState *, hipStream_t);
template hb_status launch_cg_steps<float>(int64_t, double *, double *, double *, const float *, const TilePlan &,
                                          const float *, const double *, CgWork &, CgState *, hipStream_t);

hb_status launch_residual_norm(int64_t n, const double *b, const double *t, double *r, CgWork &w, double *out,
                               hipStream_t s)
{
    const int g = vec_blocks(n);
    residual_norm_kernel<<<g, kVecThreads, 0, s>>>(n, b, t, r, nullptr, w.part_vec);
    sum_kernel<<<1, kFinThreads, 0, s>>>(w.part_vec, g, out);
    HB_HIP(hipGetLastError());
    return HB_OK;
}

hb_status launch_cg_replace(int64_t n, const double *b, const double *t, double *r, CgWork &w, CgState *st,
                            double *out, const double *inv, hipStream_t s)
{
    const int g = vec_blocks(n);
    residual_norm_kernel<<<g, kVecThreads, 0, s>>>(n, b, t, r, inv, w.part_vec);
    replace_finish_kernel<<<1, kFinThreads, 0, s>>>(w.part_vec, g, inv ? 1 : 0, st, w.rho, w.hist, out);
    HB_HIP(hipGetLastError());
    return HB_OK;
}

hb_status launch_cg_resume(CgState *st, double stop_res, hipStream_t s)
{
    resume_kernel<<<1, 64, 0, s>>>(st, stop_res);
    HB_HIP(hipGetLastError());
    return HB_OK;
}

hb_status launch_axpy(int64_t n, double *x, const double *d, hipStream_t s)
{
    axpy_kernel<<<vec_blocks(n), kVecThreads, 0, s>>>(n, x, d);
    HB_HIP(hipGetLastError());
    return HB_OK;
}

}  // namespace hb
