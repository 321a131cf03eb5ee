// Dispatch of the fused operator by polynomial degree (compile-time N) and
// workgroup shape, the schedule table behind it, and the kernel that adds the
// halo to an assembled vector.
#include <algorithm>
#include <atomic>
#include <mutex>

#include "common.h"

namespace hb {

#define HB_DECL_AX(n)                                                                                              \
    hb_status launch_ax_##n(const hb_mesh_s *, int, double, const double *, double *, double *, bool, double *,    \
                            CgState *, hipStream_t);                                                               \
    hb_status launch_ax32_##n(const hb_mesh_s *, int, double, const double *, float *, float *, double *,          \
                              CgState *, hipStream_t);                                                             \
    hb_status launch_batch_ax_##n(int, bool, const WorkItem *, int, const BatchProb *, hipStream_t);               \
    hb_status launch_ax_d_##n(const hb_mesh_s *, int, double, const double *, double *, double *, bool, double *,  \
                              CgState *, hipStream_t);                                                             \
    hb_status launch_ax32_d_##n(const hb_mesh_s *, int, double, const double *, float *, float *, double *,        \
                                CgState *, hipStream_t);                                                           \
    hb_status launch_batch_ax_d_##n(int, bool, const WorkItem *, int, const BatchProb *, hipStream_t);
HB_DECL_AX(1) HB_DECL_AX(2) HB_DECL_AX(3) HB_DECL_AX(4) HB_DECL_AX(5) HB_DECL_AX(6) HB_DECL_AX(7) HB_DECL_AX(8)
HB_DECL_AX(9) HB_DECL_AX(10) HB_DECL_AX(11) HB_DECL_AX(12) HB_DECL_AX(13) HB_DECL_AX(14) HB_DECL_AX(15)
#undef HB_DECL_AX

#define HB_ALL_N(X) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15)

namespace {

// Default entries of the schedule table.  An entry of this value means the default rule
// (ax_variant), so a caller that reads the table and writes it back changes nothing.
constexpr int kDefaultSched[2][kMaxN + 1] = {
    // N: 0  1  2  3  4  5  6  7  8  9 10 11 12 13 14 15
    {0, 1, 1, 9, 3, 1, 8, 9, 8, 29, 8, 21, 21, 5, 5, 5},  // FP64
    {0, 8, 1, 8, 1, 9, 9, 8, 9, 9, 9, 21, 0, 21, 5, 4},   // FP32
};

std::atomic<int> g_sched[2][kMaxN + 1] = {};
std::atomic<int> g_epoch{0};
std::once_flag g_init;

void init_table()
{
    std::call_once(g_init, [] {
        for (int p = 0; p < 2; ++p)
            for (int n = 0; n <= kMaxN; ++n) g_sched[p][n].store(kDefaultSched[p][n]);
    });
}

constexpr int kHaloThreads = 256;

template <typename T>
__global__ __launch_bounds__(kHaloThreads) void halo_add_kernel(TilePlan p, const T *__restrict__ halo,
                                                               T *__restrict__ y)
{
    halo_add(p, halo, y, blockIdx.x * static_cast<uint32_t>(kHaloThreads) + threadIdx.x);
}

}  // namespace

template <typename T>
hb_status launch_halo_add(const TilePlan &p, const T *halo, T *y, hipStream_t s)
{
    if (p.halo == 0) return HB_OK;
    halo_add_kernel<T><<<(p.halo + kHaloThreads - 1) / kHaloThreads, kHaloThreads, 0, s>>>(p, halo, y);
    HB_HIP(hipGetLastError());
    return HB_OK;
}
template hb_status launch_halo_add<double>(const TilePlan &, const double *, double *, hipStream_t);
template hb_status launch_halo_add<float>(const TilePlan &, const float *, float *, hipStream_t);

int ax_schedule(int N, bool fp32)
{
    init_table();
    if (N < 1 || N > kMaxN) return 0;
    return g_sched[fp32 ? 1 : 0][N].load(std::memory_order_relaxed);
}

bool ax_schedule_legal(int N, int v)
{
    const bool small = (N + 1) * (N + 1) <= 64;   // an element fits in a wave
    const bool merge = (N + 1) * (N + 1) <= 128;  // a 256-thread tile holds two or more elements
    const int lean_cols = kSchedLean | kSchedColsLds;
    const int rest = v & ~kSchedMerge;
    const bool merge_ok = merge && !(v & kSchedWave) &&
                          (!(v & (kSchedLean | kSchedThree)) || rest == (lean_cols | kSchedThree));
    return N >= 1 && N <= kMaxN && v >= 0 && v < kNumSched && (!(v & kSchedWave) || small) &&
           (!(v & kSchedLean) || !small) && (!(v & kSchedMerge) || merge_ok) &&
           (!(v & kSchedThree) || (v & lean_cols) == lean_cols);
}

void set_ax_schedule(int N, bool fp32, int v)
{
    init_table();
    g_sched[fp32 ? 1 : 0][N].store(v, std::memory_order_relaxed);
    g_epoch.fetch_add(1);
}

int ax_schedule_epoch() { return g_epoch.load(); }

hb_status launch_ax(const hb_mesh_s *m, int variant, double lambda, const double *x, double *y, double *halo,
                    bool add, double *partial, CgState *st, hipStream_t s)
{
    const bool d = (m->desc.flags & HB_MESH_DIRICHLET) != 0;
    switch (m->N) {
#define HB_CASE(n)                                                                   \
    case n:                                                                          \
        return d ? launch_ax_d_##n(m, variant, lambda, x, y, halo, add, partial, st, s) \
                 : launch_ax_##n(m, variant, lambda, x, y, halo, add, partial, st, s);
        HB_ALL_N(HB_CASE)
#undef HB_CASE
    default: return fail(HB_ERR_INVALID_ARG, "unsupported degree N");
    }
}

hb_status launch_ax32(const hb_mesh_s *m, int variant, double lambda, const double *x, float *y, float *halo,
                      double *partial, CgState *st, hipStream_t s)
{
    if (!m->tab32) return fail(HB_ERR_INVALID_ARG, "the FP32 operator needs a mesh built with HB_MESH_FP32");
    const bool d = (m->desc.flags & HB_MESH_DIRICHLET) != 0;
    switch (m->N) {
#define HB_CASE(n)                                                                \
    case n:                                                                       \
        return d ? launch_ax32_d_##n(m, variant, lambda, x, y, halo, partial, st, s) \
                 : launch_ax32_##n(m, variant, lambda, x, y, halo, partial, st, s);
        HB_ALL_N(HB_CASE)
#undef HB_CASE
    default: return fail(HB_ERR_INVALID_ARG, "unsupported degree N");
    }
}

hb_status launch_ax_full(const hb_mesh_s *m, double lambda, const double *x, double *y, double *halo, bool add,
                         hipStream_t s)
{
    const int v = mesh_variant(m, false);  // read once: another thread may set the table between the launches
    const hb_status st = launch_ax(m, v, lambda, x, y, halo, add, nullptr, nullptr, s);
    return st ? st : launch_halo_add(m->plan[v], halo, y, s);
}

hb_status launch_ax_full(const hb_mesh_s *m, double lambda, const double *x, float *y, float *halo, hipStream_t s)
{
    const int v = mesh_variant(m, true);
    const hb_status st = launch_ax32(m, v, lambda, x, y, halo, nullptr, nullptr, s);
    return st ? st : launch_halo_add(m->plan[v], halo, y, s);
}

hb_status launch_batch_ax(int N, int variant, bool fp32, bool dirichlet, const WorkItem *items, int nitems,
                          const BatchProb *probs, hipStream_t s)
{
    switch (N) {
#define HB_CASE(n)                                                                                   \
    case n:                                                                                          \
        return dirichlet ? launch_batch_ax_d_##n(variant, fp32, items, nitems, probs, s)             \
                         : launch_batch_ax_##n(variant, fp32, items, nitems, probs, s);
        HB_ALL_N(HB_CASE)
#undef HB_CASE
    default: return fail(HB_ERR_INVALID_ARG, "unsupported degree N");
    }
}

hb_status launch_batch_any64(const WorkItem *, int, size_t, const BatchProb *, hipStream_t);
hb_status launch_batch_any32(const WorkItem *, int, size_t, const BatchProb *, hipStream_t);
hb_status launch_batch_any64_d(const WorkItem *, int, size_t, const BatchProb *, hipStream_t);
hb_status launch_batch_any32_d(const WorkItem *, int, size_t, const BatchProb *, hipStream_t);
hb_status launch_batch_ax_any(bool fp32, bool dirichlet, const WorkItem *items, int nitems, size_t lds,
                              const BatchProb *probs, hipStream_t s)
{
    if (nitems == 0) return HB_OK;
    return fp32 ? (dirichlet ? launch_batch_any32_d : launch_batch_any32)(items, nitems, lds, probs, s)
                : (dirichlet ? launch_batch_any64_d : launch_batch_any64)(items, nitems, lds, probs, s);
}

int variant_epb(int N, int variant)
{
    const int np2 = (N + 1) * (N + 1), target = variant == 1 && np2 <= 64 ? 64 : 256;
    return std::max(target / np2, 1);
}

int default_schedule(int N, bool fp32) { return kDefaultSched[fp32 ? 1 : 0][N]; }

int default_variant(int N, int64_t elements)
{
    return (N + 1) * (N + 1) <= 64 && elements < static_cast<int64_t>(kSmallLaunch) * variant_epb(N, 0) ? 1 : 0;
}

int ax_variant(int N, bool fp32, int64_t elements)
{
    if ((N + 1) * (N + 1) > 64) return 0;
    const int sched = ax_schedule(N, fp32);
    if (sched != default_schedule(N, fp32)) return sched & kSchedWave ? 1 : 0;
    return default_variant(N, elements);
}

int mesh_variant(const hb_mesh_s *m, bool fp32)
{
    if (m->desc.flags & HB_MESH_GATHER) return default_variant(m->N, m->E);  // reproducible whatever the table holds
    return ax_variant(m->N, fp32, m->E);
}

int ax_blocks_max(const hb_mesh_s *m) { return std::max(m->plan[0].tiles(), m->plan[1].tiles()); }

}  // namespace hb
