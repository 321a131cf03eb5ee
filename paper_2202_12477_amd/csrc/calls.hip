// Who has which halo, and the operator calls of the C ABI (hb_ax and its forms).
//
// A call is two launches with a halo between them, and the caller orders neither calls on
// different streams nor the replays of graphs that calls were captured into.  So every
// stream's calls have a halo, and every capture's, for as long as the graph lives; host
// threads that call on the same mesh take turns for the length of a call's two launches.
// The solves on a mesh, which the caller serialises, have one.  The mesh's own halo, part of
// its allocation, is the solves' or a stream's, whoever asks first; the others are allocated
// then (with two in the mesh, creating 32^3 N = 7 took 57 us longer).  A small y += A x is
// one launch that adds atomically, and needs none of this.
#include <new>

#include "common.h"

namespace hb {
namespace {

// Streams that a mesh keeps halos for; the next new one waits for the device and takes
// one of theirs (a framework's pool of streams is about 32).
constexpr int kCallStreams = 64;

// y += A x in one launch, each sum added to y atomically, up to so many local nodes; above,
// the atomics take longer than a second launch.  Against the two launches: 4^3 N = 3 7.8 us
// against 11.3, 10^3 N = 7 10.5 against 14.6, 14^3 N = 7 (1.4 million nodes) 19.2 against
// 21.6, 16^3 (2.1 million) 27.4 against 23.6; 16^3 N = 6 (1.4) 19.9 against 21.9, 20^3 (2.7)
// 33.7 against 29.1; 10^3 N = 9 (1.0) 17.6 against 20.8, 12^3 (1.7) 28.5 both.
constexpr int64_t kDirectNodes = 3 << 19;

// hipMalloc that disturbs no capture: on a thread that captures, or beside another that does.
hb_status alloc_halo(hb_mesh_s *m, double **mem)
{
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    const bool swapped = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
    const hb_status st = dev_alloc(mem, m->halo_len, &m->device_bytes);
    if (swapped) (void)hipThreadExchangeStreamCaptureMode(&mode);
    return st;
}

// `live` of a capture's halo is cleared when the graph and its executables are gone; if
// that cannot be arranged, the halo stays the capture's until the mesh goes.
std::shared_ptr<std::atomic<bool>> with_graph(hipGraph_t graph)
{
    using Flag = std::shared_ptr<std::atomic<bool>>;
    Flag live = std::make_shared<std::atomic<bool>>(true);
    auto *ref = new Flag(live);
    hipUserObject_t obj = nullptr;
    auto gone = [](void *p) {
        Flag *f = static_cast<Flag *>(p);
        (*f)->store(false, std::memory_order_release);
        delete f;
    };
    if (hipUserObjectCreate(&obj, ref, gone, 1, hipUserObjectNoDestructorSync) != hipSuccess) {
        (void)hipGetLastError();
        delete ref;
    } else if (hipGraphRetainUserObject(graph, obj, 1, hipGraphUserObjectMove) != hipSuccess) {
        (void)hipGetLastError();
        live = std::make_shared<std::atomic<bool>>(true);
        (void)hipUserObjectRelease(obj, 1);
    }
    return live;
}

// The halo of a call on stream s (call_mu is held); without `allocate` one of another
// stream's is taken after waiting for the device.
hb_status call_halo(hb_mesh_s *m, hipStream_t s, bool allocate, double **out)
{
    if (m->halo_len == 0) {  // no tile has a neighbour
        *out = m->own_halo;
        return HB_OK;
    }
    unsigned long long id = 0;
    hipGraph_t graph = nullptr;
    if (s != nullptr && s != hipStreamLegacy) {  // (those cannot be captured)
        hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
        if (hipStreamGetCaptureInfo_v2(s, &status, &id, &graph, nullptr, nullptr) != hipSuccess) (void)hipGetLastError();
        if (status != hipStreamCaptureStatusActive) id = 0;
    }
    const std::thread::id thread = s == hipStreamPerThread ? std::this_thread::get_id() : std::thread::id();
    CallHalo *take = nullptr;
    int streams = 0;
    for (CallHalo &h : m->call_halo) {
        if (h.capture && !h.live->load(std::memory_order_acquire)) h.used = false;
        if (!h.used) {  // (no capture takes the mesh's own: lease_halo counts on it)
            if (!take && (id == 0 || h.mem != m->own_halo)) take = &h;
        } else if (h.stream == s && h.capture == id && h.thread == thread) {
            *out = h.mem;
            return HB_OK;
        } else {
            streams += h.capture == 0;
        }
    }
    hb_status st = HB_OK;
    if (!take && allocate && (id != 0 || streams < kCallStreams)) {
        CallHalo h;
        m->call_halo.reserve(m->call_halo.size() + 1);
        if ((st = alloc_halo(m, &h.mem)) == HB_OK) {
            m->call_halo.push_back(std::move(h));
            take = &m->call_halo.back();
        }
    }
    if (!take && id == 0 && streams > 0) {
        HB_HIP(hipDeviceSynchronize());
        for (CallHalo &h : m->call_halo)
            if (h.capture == 0) {
                h.used = false;
                take = &h;
            }
    }
    if (!take) return st ? st : fail(HB_ERR_OUT_OF_MEMORY, "no halo without an allocation");
    if (id != 0) take->live = with_graph(graph);
    take->used = true;
    take->stream = s;
    take->thread = thread;
    take->capture = id;
    *out = take->mem;
    return HB_OK;
}

// The solves have a halo, or take the mesh's own if no stream has it (call_mu is held).
bool own_for_solves(hb_mesh_s *m)
{
    if (!m->halo && !m->call_halo.empty() && m->call_halo[0].mem == m->own_halo && !m->call_halo[0].used) {
        m->call_halo.erase(m->call_halo.begin());
        m->halo = m->own_halo;
    }
    if (!m->halo && m->halo_len == 0) m->halo = m->own_halo;
    return m->halo != nullptr;
}

template <typename F>
hb_status with_call_halo(hb_mesh_s *m, hipStream_t s, F &&launch)
{
    try {
        std::lock_guard<std::mutex> lock(m->call_mu);
        double *halo = nullptr;
        const hb_status st = call_halo(m, s, true, &halo);
        return st ? st : launch(halo);
    } catch (const std::bad_alloc &) {
        return fail(HB_ERR_OUT_OF_MEMORY, "operator call: host allocation failed");
    }
}

}  // namespace

hb_status call_ax(hb_mesh_s *m, double lambda, const double *x, double *y, bool add, hipStream_t s)
{
    if (add && m->NL <= kDirectNodes && !(m->desc.flags & HB_MESH_GATHER))
        return launch_ax(m, mesh_variant(m, false), lambda, x, y, nullptr, true, nullptr, nullptr, s);
    return with_call_halo(m, s, [&](double *halo) { return launch_ax_full(m, lambda, x, y, halo, add, s); });
}

hb_status ensure_solve_halo(hb_mesh_s *m)
{
    std::lock_guard<std::mutex> lock(m->call_mu);
    return own_for_solves(m) ? HB_OK : alloc_halo(m, &m->halo);
}

hb_status lease_halo(hb_mesh_s *m, hipStream_t s, HaloLease *lease)
{
    try {
        lease->lock = std::unique_lock<std::mutex>(m->call_mu);
        if (!own_for_solves(m)) return call_halo(m, s, false, &lease->halo);
        lease->halo = m->halo;
        lease->lock.unlock();
        return HB_OK;
    } catch (const std::bad_alloc &) {
        return fail(HB_ERR_OUT_OF_MEMORY, "host allocation failed");
    }
}

hb_status call_ax32(hb_mesh_s *m, double lambda, const double *x, float *y, hipStream_t s)
{
    return with_call_halo(m, s, [&](double *halo) {
        return launch_ax_full(m, lambda, x, y, reinterpret_cast<float *>(halo), s);
    });
}

}  // namespace hb
