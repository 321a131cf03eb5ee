// Internal declarations shared by the HIP translation units of libhbmi.
// Not installed; the public interface is include/hbmi.h.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstddef>
#include <cstdint>
#include <memory>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

#include "hbmi.h"
#include "tile.h"

namespace hb {

constexpr int kMaxN = 15;
// Bits of the schedule table's entries.  The operator has two workgroup shapes
// (variants), 256 threads and one wave: an explicitly set entry selects the
// one-wave shape by kSchedWave, where an element fits a wave (N <= 7); the other
// bits name values the table accepts and do not change the kernel.
constexpr int kSchedColsLds = 1, kSchedWave = 2, kSchedLean = 4, kSchedMerge = 8, kSchedThree = 16,
              kNumSched = 32;
constexpr int kGeo = 7;  // G_rr, G_rs, G_rt, G_ss, G_st, G_tt, c

// Thread-local error message behind hb_last_error().
void set_error(const std::string &msg);
hb_status fail(hb_status st, const std::string &msg);
hb_status hip_fail(hipError_t err, const char *what);

// Device allocation that reports HB_ERR_OUT_OF_MEMORY and adds to *tally.
template <typename T>
inline hb_status dev_alloc(T **p, size_t count, size_t *tally)
{
    if (hipMalloc(reinterpret_cast<void **>(p), sizeof(T) * count) != hipSuccess) {
        (void)hipGetLastError();
        *p = nullptr;
        return fail(HB_ERR_OUT_OF_MEMORY, "device allocation of " + std::to_string(sizeof(T) * count) + " bytes failed");
    }
    *tally += sizeof(T) * count;
    return HB_OK;
}

#define HB_HIP(call)                                      \
    do {                                                  \
        hipError_t err_ = (call);                         \
        if (err_ != hipSuccess) return hb::hip_fail(err_, #call); \
    } while (0)

// Device-resident state of one CG solve (Algorithm 1).  Scalars never leave
// the device and no kernel takes the iteration number as an argument, so one
// captured iteration can be replayed and problems at different iterations can
// share launches.  Fields are written only by single-block kernels and read by
// later kernels:
//   alpha (first single-block kernel of an iteration): turns `pending` into
//     `done`, else advances `it` and computes alpha (or sets `broke` on breakdown,
//     which the update step turns into `done`: no launch writes a field that its
//     own blocks still branch on);
//   beta: records rho_{it+1}, beta, the history and `iters`; a stop decided
//     here only sets `pending`, so this iteration's update still runs.
// Every streaming kernel returns at once when `done` is set (an operator call
// issued after `pending` was set is wasted but harmless: it touches only Ap).
struct CgState {
    double bb;         // b . b
    double alpha;      // alpha of the current iteration
    double beta;       // beta of the current iteration
    double pAp;        // p . A p of the current iteration
    double rho;        // r.r (r.z with the Jacobi preconditioner) after the completed iterations
    double rho_j;      // the same at the start of the current iteration
    double rtol;       // < 0 in fixed-iteration mode
    double stop_res;   // stop once ||r_j|| <= stop_res (< 0: never; set from rtol ||b|| at the start)
    int32_t max_iter;
    int32_t it;        // index of the current iteration (-1 before the first)
    int32_t iters;     // completed iterations
    int32_t done;      // no further kernel of this solve does anything
    int32_t pending;   // stop after the current iteration's update
    int32_t status;    // hb_status of the solve
    int32_t broke;     // breakdown in the current iteration: its remaining steps do nothing
};

// One problem of a batched solve, as the batched kernels see it (device copy).
struct BatchProb {
    const double *coef;   // the elements' trilinear maps
    double *halo;         // operator outputs on DOFs of neighbouring tiles (halo32: the same memory)
    float *halo32;
    double lambda;
    double *x, *r, *p, *Ap;
    float *Ap32;
    double *rho, *hist, *part_ax, *part_vec;
    CgState *st;
    int64_t E, NG;
    int32_t N, ax_tiles, vec_chunks, use32;  // use32: the operator of this problem is the FP32 one
    int32_t dirichlet;                       // a Dirichlet box (host side: its class of operator launches)
    const double *inv;                       // Jacobi: 1 / diag(A) (nullptr: no preconditioner)
    const double *tab, *xw;                  // the degree's tables
    const float *tab32;
    int32_t variant;                         // the operator's workgroup shape, and its tiles
    TilePlan plan;
};

// A unit of batched work: problem index and tile (operator) or chunk (vectors).
struct WorkItem {
    int32_t prob, idx;
};

// The persistent batched launch (persist.hip): workgroup -> (problem, rank
// among the problem's workgroups), and per problem its workgroup count, its
// iteration budget for the launch and its operator tiles.
struct PersistWg {
    int32_t prob, rank;
};
struct PersistSlot {
    TilePlan plan;
    int32_t nwg, iters;
};

// Per-mesh CG workspace (device), allocated on first use.
struct CgWork {
    int64_t n = 0;         // N_G it was sized for
    int32_t hist_len = 0;  // entries in hist
    double *r = nullptr, *p = nullptr, *Ap = nullptr;
    double *part_ax = nullptr;  // operator block partials of p.Ap (>= operator grid)
    double *part_vec = nullptr; // vector-kernel block partials (>= 2 * vector grid)
    int32_t part_ax_len = 0, part_vec_len = 0;
    double *rho = nullptr;      // r_j . r_j (r_j . z_j with the Jacobi preconditioner), j = 0..max_iter
    // mixed-precision refinement: outer residual, correction, FP32 operator output
    double *rout = nullptr, *d = nullptr;
    float *Ap32 = nullptr;
    double *halo = nullptr;     // of the solve's operators (not the workspace's own)
    double *hist = nullptr;     // ||r_j||, j = 0..max_iter
    CgState *state = nullptr;
    double *dnorm = nullptr;        // one device scalar (a squared norm)
    CgState *host_state = nullptr;  // pinned mirror for read-back
    double *host_norm = nullptr;    // pinned mirror of dnorm
    size_t bytes = 0;               // device bytes held (counted in the mesh's device_bytes)
    // captured iteration graphs (hb_cg_opts.graph_k), keyed by their arguments
    struct Graph {
        hipGraphExec_t exec = nullptr;
        int elem = 0;   // bytes per operator output entry (8: FP64 operator, 4: FP32)
        int epoch = 0;  // schedule-table version the kernels were captured under
        int k = 0;
        double lambda = 0.0;
        const void *x = nullptr, *Ap = nullptr;
        bool pc = false;  // Jacobi-preconditioned iteration
    };
    Graph graphs[2];
    int graph_next = 0;
    int graph_k = 0;           // the current solve's graph length (0: plain launches)
    hipStream_t cap = nullptr; // private stream the graphs are captured on
    // Jacobi preconditioner: 1 / diag(A) for lambda = jlambda (allocated on first use)
    double *jinv = nullptr;
    double jlambda = 0.0;
    bool jvalid = false;
    bool pc = false;           // the current solve is preconditioned (iterations use jinv)
};

// A halo of the operator calls (hb_ax and its forms).  A call's operator writes the halo
// and its second launch adds it, so calls that may overlap on the device take one each:
// a stream's calls one, the calls captured from a stream into a graph another, which may
// be replayed at any time on any stream (calls.hip).
struct CallHalo {
    double *mem = nullptr;
    bool used = false;
    hipStream_t stream = nullptr;
    std::thread::id thread;          // set for hipStreamPerThread, one handle for a stream to each thread
    unsigned long long capture = 0;  // 0: of calls that run at once
    std::shared_ptr<std::atomic<bool>> live;  // a capture's: false once its graph and the graph's executables are gone
};

}  // namespace hb

// Global nodes (DOFs) of a box mesh: every GLL node of the box, or only the
// interior ones with HB_MESH_DIRICHLET.
inline int64_t box_global_nodes(const hb_mesh_desc &d)
{
    const int64_t gx = (int64_t)d.nx * d.N + 1, gy = (int64_t)d.ny * d.N + 1, gz = (int64_t)d.nz * d.N + 1;
    return (d.flags & HB_MESH_DIRICHLET) ? (gx - 2) * (gy - 2) * (gz - 2) : gx * gy * gz;
}

struct hb_mesh_s {
    hb_mesh_desc desc;
    int N = 0;
    int64_t E = 0, NL = 0, NG = 0;
    // what the operator reads (setup.hip), in one allocation: 21 coefficients per
    // element of its trilinear map, the half matrices of D in FP64 and (HB_MESH_FP32)
    // FP32, the GLL nodes and weights in one array, and D, [(N+1)^2] row-major
    unsigned char *mem = nullptr;
    double *coef = nullptr, *D = nullptr;
    double *tab = nullptr, *xw = nullptr;
    float *tab32 = nullptr;
    hb::TilePlan plan[2];      // the tiles of each workgroup shape
    // operator outputs on DOFs of neighbouring tiles: of the solves, and of the operator
    // calls (FP64 and FP32 operators of one user run in turn and share the memory).  The
    // mesh's allocation holds one, for the first that asks (calls.hip).  Under call_mu,
    // with device_bytes.
    size_t halo_len = 0;
    double *own_halo = nullptr, *halo = nullptr;  // the mesh's; the solves' (nullptr: none yet)
    std::mutex call_mu;
    std::vector<hb::CallHalo> call_halo;
    double h_xi[hb::kMaxN + 1], h_w[hb::kMaxN + 1], h_D[(hb::kMaxN + 1) * (hb::kMaxN + 1)];
    hb::CgWork cg;
    size_t device_bytes = 0;
};

namespace hb {

// Host-side 1D basis (basis.cpp): GLL nodes ascending, weights, D[i][j] = l_j'(xi_i).
void gll_basis(int N, double *xi, double *w, double *D);

// Setup (setup.hip): plans, tables, element maps and halos (after the host basis is
// known), and the check of the Jacobian; waits for the stream.
hb_status build_mesh(hb_mesh_s *m, hipStream_t s);
// Z and the geometric factors to host arrays, [E][(N+1)^3] and [E][7][(N+1)^3] (either
// may be null); waits.
hb_status export_geometry(const hb_mesh_s *m, double *host_geo, int32_t *host_map);
hb_status launch_rhs(int64_t n, uint64_t seed, double *b, hipStream_t s);

// Operator (ax*.hip).  y = A x (add: y += A x) on the DOFs each tile owns, the
// rest of the tiles' outputs in the mesh's halo: whoever reads y next adds
// halo_sum (tile.h).  With st != nullptr this is the operator step of CG: it
// returns at once if the solve is done, and each block also writes its share of
// x . A x to partial[block].  halo: the mesh's, or a call's; y += A x without one adds
// all of it to y, atomically.
// variant: the workgroup shape, so the tiles (mesh_variant, asked once for the launches
// that belong together: the table behind it may be set meanwhile).
hb_status launch_ax(const hb_mesh_s *m, int variant, double lambda, const double *x, double *y, double *halo,
                    bool add, double *partial, CgState *st, hipStream_t s);
// The FP32 operator (mesh built with HB_MESH_FP32): x FP64, y and its halo FP32.
hb_status launch_ax32(const hb_mesh_s *m, int variant, double lambda, const double *x, float *y, float *halo,
                      double *partial, CgState *st, hipStream_t s);
// y += the halo of these tiles.
template <typename T>
hb_status launch_halo_add(const TilePlan &p, const T *halo, T *y, hipStream_t s);
// y = A x (add: y += A x), complete: the operator, then the halo added.
hb_status launch_ax_full(const hb_mesh_s *m, double lambda, const double *x, double *y, double *halo, bool add,
                         hipStream_t s);
hb_status launch_ax_full(const hb_mesh_s *m, double lambda, const double *x, float *y, float *halo, hipStream_t s);
// The same as a caller's own operation, from any thread and on any stream, beside other
// calls and a solve on the mesh: with a halo that no call it may overlap uses (calls.hip).
hb_status call_ax(hb_mesh_s *m, double lambda, const double *x, double *y, bool add, hipStream_t s);
hb_status call_ax32(hb_mesh_s *m, double lambda, const double *x, float *y, hipStream_t s);
// A halo for the mesh's solves (m->halo), before the first one.
hb_status ensure_solve_halo(hb_mesh_s *m);
// A halo for one synchronous solve on stream s, without an allocation: the solves' if they
// have or can have one, else an operator call's, and such calls wait while it is held.
struct HaloLease {
    double *halo = nullptr;
    std::unique_lock<std::mutex> lock;
};
hb_status lease_halo(hb_mesh_s *m, hipStream_t s, HaloLease *lease);
// The memory the mesh holds changed by `bytes`.
inline void count_bytes(hb_mesh_s *m, ptrdiff_t bytes)
{
    std::lock_guard<std::mutex> lock(m->call_mu);
    m->device_bytes += bytes;
}
// The most operator blocks (tiles) of a mesh in any variant (sizes partials).
int ax_blocks_max(const hb_mesh_s *m);
// Elements of a workgroup of a variant.
int variant_epb(int N, int variant);
// The autotuner (tune.hip): time each workgroup shape of a class on a synthetic
// box of about local_nodes local nodes and install the faster; the cached
// form tunes each (degree, precision, power-of-two size class) once per
// process and installs its winner on later calls.
hb_status tune_class(int N, bool fp32, int64_t local_nodes, int reps, hb_tune_result *out, hipStream_t s);
int tune_size_class(int64_t local_nodes);
hb_status tune_class_cached(int N, bool fp32, int64_t local_nodes, hipStream_t s, int *schedule);
// The variant of a launch over `elements` elements: the schedule table's if the
// class's entry is not the default; else 256-thread workgroups, or one-wave workgroups
// where fewer than kSmallLaunch of the former would run (a launch that leaves
// compute units idle is bound by latency, and more, smaller workgroups finish
// sooner).  mesh_variant: of a single-problem launch on this mesh.
constexpr int kSmallLaunch = 256;
int ax_variant(int N, bool fp32, int64_t elements);
int default_variant(int N, int64_t elements);  // as with the default entry
int default_schedule(int N, bool fp32);
int mesh_variant(const hb_mesh_s *m, bool fp32);
// Schedule table (per degree and precision), shared by every solve path.
int ax_schedule(int N, bool fp32);
bool ax_schedule_legal(int N, int sched);
void set_ax_schedule(int N, bool fp32, int sched);
int ax_schedule_epoch();

// Vector kernels of CG (cg.hip).  TAp is the type of the operator output Ap
// (double for the FP64 operator, float for the FP32 one); every other vector
// and every dot product is FP64.
int vec_blocks(int64_t n);
hb_status launch_zero(double *v, int64_t n, hipStream_t s);
hb_status launch_zero(float *v, int64_t n, hipStream_t s);
hb_status launch_cg_setup_state(CgState *st, int max_iter, double rtol, hipStream_t s);
template <typename TAp>
hb_status launch_cg_init(int64_t n, const double *b, double *x, double *r, double *p, TAp *Ap, int x0_zero,
                         CgWork &w, CgState *st, hipStream_t s);
// Where each block of the residual (update) step sums the operator's (the
// residual's) partials itself, an iteration is three launches instead of five.
// Every block reads all partials, so only while they are few: a single-block
// launch takes about 5 us with its gap, 2048 partials 1 us more in each block.
constexpr int kFuseMax = 2048;

// The steps of an iteration after the operator: alpha, r -= alpha Ap with r.r, beta,
// x += alpha p and p = r + beta p (inv: the Jacobi inverse diagonal).
template <typename TAp>
hb_status launch_cg_steps(int64_t n, double *x, double *p, double *r, const TAp *Ap, const TilePlan &plan,
                          const TAp *halo, const double *inv, CgWork &w, CgState *st, hipStream_t s);
// alpha, residual, beta and update in one workgroup, for vectors of at most
// kCgTailMax entries: two launches per iteration.  Measured per iteration at 2197 DOFs:
// 12.2 us against 15.5 us with the three launches; the whole iteration in one
// workgroup, operator included, took 18 us (one compute unit's arithmetic).
constexpr int64_t kCgTailMax = 4096;
template <typename TAp>
hb_status launch_cg_tail(int64_t n, double *x, double *p, double *r, const TAp *Ap, const TilePlan &plan,
                         const TAp *halo, const double *inv, CgWork &w, CgState *st, hipStream_t s);
// 1 / diag(A) into inv (Jacobi preconditioner), for the mesh's operator at lambda; every
// sum in a fixed order (through the halo).
hb_status launch_jacobi_inverse(const hb_mesh_s *m, double lambda, double *inv, double *halo, hipStream_t s);
// Residual replacement after the completed iterations: r = b - t (t = A x
// from the FP64 operator), rho_iters = r.r (r.z with the Jacobi inverse
// diagonal inv), history entry iters = ||r||, *out = r.r; then the solve
// resumes with a new stopping threshold on ||r||.
hb_status launch_cg_replace(int64_t n, const double *b, const double *t, double *r, CgWork &w, CgState *st,
                            double *out, const double *inv, hipStream_t s);
hb_status launch_cg_resume(CgState *st, double stop_res, hipStream_t s);
// Refinement helpers: r = b - t with ||r||^2 into *out (one block finishes), and x += d.
hb_status launch_residual_norm(int64_t n, const double *b, const double *t, double *r, CgWork &w, double *out,
                               hipStream_t s);
hb_status launch_axpy(int64_t n, double *x, const double *d, hipStream_t s);

// Chunks of the batched and fused vector steps: kVecChunk entries, four per thread
// (4096-entry chunks ran the 64-problem batch 6% slower).
constexpr int kVecChunk = 1024;
__host__ __device__ inline int vec_chunks(int64_t n) { return static_cast<int>((n + kVecChunk - 1) / kVecChunk); }
// Partial sums the vector steps of a mesh write (two per chunk when preconditioned).
inline int64_t vec_partials(const hb_mesh_s *m)
{
    return std::max<int64_t>(3 * vec_blocks(m->NG), 2 * static_cast<int64_t>(vec_chunks(m->NG)));
}

// Batched kernels (batch.hip).
// variant: the class's workgroup shape (the one its work list was built for);
// dirichlet: the class's problems are Dirichlet boxes.
hb_status launch_batch_ax(int N, int variant, bool fp32, bool dirichlet, const WorkItem *items, int nitems,
                          const BatchProb *probs, hipStream_t s);
// The same for problems of several degrees in one launch, a workgroup to each item in the
// list's order; lds: the largest of their shapes' (batch_ax_lds).
hb_status launch_batch_ax_any(bool fp32, bool dirichlet, const WorkItem *items, int nitems, size_t lds,
                              const BatchProb *probs, hipStream_t s);
size_t batch_ax_lds(int N, int variant, bool fp32);
// The steps after the operator over the problems of a list (plist, np) and their
// chunks (items, nitems); fused: no problem has more than kFuseMax partials.
hb_status launch_batch_steps(const int32_t *plist, int np, const WorkItem *items, int nitems, const BatchProb *probs,
                             bool fused, hipStream_t s);

// The persistent batched launch (persist.hip): every running problem advances
// up to slots[p].iters iterations inside one cooperative launch of `nwg`
// workgroups, each problem on its own workgroups (wgs), synchronised by
// per-problem barriers over the counters bar[p] (zero before the launch).  A
// barrier wait that exceeds its spin limit sets *err and ends the launch.
// Degrees the kernel is compiled for, its workgroup size, and how many of its
// workgroups the device holds at once (0 if it cannot be launched).
bool persist_degree(int N);
constexpr int kPersistThreads = 256;
int persist_capacity();
int persist_spread();  // workgroups beyond one to a problem: up to so many in all (the compute units)
hb_status launch_batch_persistent(bool dirichlet, const PersistWg *wgs, int nwg, const PersistSlot *slots,
                                  const BatchProb *probs, uint32_t *bar, int32_t *err, hipStream_t s);

// 8:1 streaming probe (stream.hip).
hb_status launch_stream_probe(const double *in, double *out, int64_t n, hipStream_t s);

}  // namespace hb
