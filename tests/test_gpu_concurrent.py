"""Calls that meet: the schedule table set by one host thread while another works; operator
calls on one mesh from several streams, threads and graphs, each with its own x and y.
Every sum of the operator has a fixed order, so results that met nothing are the same bits."""
import ctypes
import os
import sys
import threading

import numpy as np
import pytest

import inputs
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2202_12477_amd as hb  # noqa: E402

DEV = torch.device("cuda:0")


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy().astype(np.float64)


def relerr(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("nx,ny,nz,N", [(9, 7, 5, 3), (5, 3, 4, 7)])
def test_table_set_while_calls_run(nx, ny, nz, N):
    """A call's launches work on one set of tiles, whenever another thread sets the table:
    y = A x and y = A_32 x within the bounds of the other operator tests (1e-12, 2e-5), a
    fixed CG solve within 1e-9 of the undisturbed one (as other schedules' solves)."""
    say(f"[case] table set meanwhile {nx}x{ny}x{nz} N={N}")
    precs = (hb.PREC_FP64, hb.PREC_FP32_RR)
    saved = {p: hb.get_schedule(N, p) for p in precs}
    m = hb.Mesh(nx, ny, nz, N, jitter=0.1, seed=N, fp32=True)
    ref = oracle.Mesh(nx, ny, nz, N, jitter=0.1, seed=N)
    x = torch.as_tensor(inputs.random_vector(m.NG, 70 + N), device=DEV)
    yr = ref.ax(host(x), 1.3)
    sol = torch.empty_like(x)
    m.cg(1.3, x, sol, max_iter=30)
    stop = threading.Event()

    def setter():
        v = 0
        while not stop.is_set():
            v ^= 2
            for p in precs:
                hb.set_schedule(N, p, v)

    t = threading.Thread(target=setter)
    t.start()
    try:
        ys = [torch.empty_like(x) for _ in range(200)]
        y32 = [torch.empty(m.NG, dtype=torch.float32, device=DEV) for _ in range(200)]
        for a, b in zip(ys, y32):
            m.ax(1.3, x, a)
            m.ax_f32(1.3, x, b)
        sols = [torch.empty_like(x) for _ in range(20)]
        for s in sols:
            m.cg(1.3, x, s, max_iter=30)
    finally:
        stop.set()
        t.join()
        for p, v in saved.items():
            hb.set_schedule(N, p, v)
    assert max(relerr(host(y), yr) for y in ys) <= 1e-12
    assert max(relerr(host(y), yr) for y in y32) <= 2e-5
    assert max(relerr(host(s), host(sol)) for s in sols) <= 1e-9
    m.close()


@pytest.fixture
def meet():
    """A mesh whose operator takes long enough for calls to overlap, and vectors with their
    undisturbed results."""
    m = hb.Mesh(17, 15, 14, 7, jitter=0.1, seed=2, fp32=True)
    xs = [torch.as_tensor(inputs.random_vector(m.NG, 90 + i), device=DEV) for i in range(4)]
    ys = [m.ax(1.3, x, torch.empty_like(x)) for x in xs]
    torch.cuda.synchronize()
    yield m, xs, ys
    m.close()


def out_like(x, n):
    return [torch.full_like(x, float("nan")) for _ in range(n)]


def test_calls_on_two_streams(meet):
    say("[case] two streams, one host thread")
    m, xs, ys = meet
    streams = [torch.cuda.Stream() for _ in range(3)]
    y32 = m.ax_f32(1.3, xs[2], torch.empty(m.NG, dtype=torch.float32, device=DEV))
    got = [out_like(xs[0], 40), out_like(xs[0], 40), [torch.empty_like(y32) for _ in range(40)]]
    added = [torch.zeros_like(x) for x in xs[:2]]
    torch.cuda.synchronize()
    for k in range(40):
        for i in range(2):
            m.ax(1.3, xs[i], got[i][k], stream=streams[i])
            m.ax_add(1.3, xs[i], added[i], stream=streams[i])
        m.ax_f32(1.3, xs[2], got[2][k], stream=streams[2])
    torch.cuda.synchronize()
    for i in range(2):
        assert all(torch.equal(y, ys[i]) for y in got[i])
        assert relerr(host(added[i]), 40.0 * host(ys[i])) <= 1e-12
    assert all(torch.equal(y, y32) for y in got[2])


@pytest.mark.parametrize("prec", [hb.PREC_FP64, hb.PREC_FP32_RR])
def test_threads_on_one_stream_beside_a_solve(meet, prec):
    say(f"[case] three threads on one stream, a solve among them, prec={prec}")
    m, xs, ys = meet
    kw = dict(max_iter=40) if prec == hb.PREC_FP64 else dict(max_iter=4000, fixed_iters=False, rtol=1e-8, prec=prec)
    m.cg(1.3, xs[3], want := torch.empty_like(xs[3]), **kw)
    got = [out_like(xs[0], 60), out_like(xs[0], 60)]
    sols = out_like(xs[3], 4)
    stream = torch.cuda.current_stream()
    torch.cuda.synchronize()

    def work(i):
        for y in got[i]:
            m.ax(1.3, xs[i], y, stream=stream)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for s in sols:
        m.cg(1.3, xs[3], s, stream=stream, **kw)
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for i in range(2):
        assert all(torch.equal(y, ys[i]) for y in got[i])
    assert all(torch.equal(s, want) for s in sols)


def test_captured_calls_replayed_beside_others(meet):
    """Two graphs captured on one stream, replayed on two others beside eager calls on a
    third; then the graphs are dropped and captured anew."""
    m, xs, ys = meet
    side = torch.cuda.Stream()
    streams = [torch.cuda.Stream() for _ in range(3)]
    for again in range(3):
        say(f"[case] captured calls, capture {again}")
        got = out_like(xs[0], 3)
        graphs = []
        for i in range(2):
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=side):
                m.ax(1.3, xs[i], got[i])
            graphs.append(g)
        torch.cuda.synchronize()
        for rep in range(4):
            for y in got:
                y.fill_(float("nan"))
            torch.cuda.synchronize()
            for k in range(10):
                for i in range(2):
                    with torch.cuda.stream(streams[i]):
                        graphs[i].replay()
                m.ax(1.3, xs[2], got[2], stream=streams[2])
                m.ax(1.3, xs[3], out_like(xs[3], 1)[0])
            torch.cuda.synchronize()
            assert all(torch.equal(got[i], ys[i]) for i in range(3))
        del graphs, g


def test_more_streams_than_a_mesh_keeps_halos_for(meet):
    say("[case] 70 streams")
    m, xs, ys = meet
    hip = ctypes.CDLL(os.path.join(os.path.dirname(torch.__file__), "lib", "libamdhip64.so"))
    streams = []
    for _ in range(70):
        s = ctypes.c_void_p()
        assert hip.hipStreamCreateWithFlags(ctypes.byref(s), 1) == 0  # non-blocking
        streams.append(s)
    small = hb.Mesh(5, 4, 3, 3, jitter=0.1, seed=4)
    x = torch.as_tensor(inputs.random_vector(small.NG, 95), device=DEV)
    want = small.ax(1.3, x, torch.empty_like(x))
    got = out_like(x, 140)
    torch.cuda.synchronize()
    for k, y in enumerate(got):
        small.ax(1.3, x, y, stream=streams[k % 70].value)
    torch.cuda.synchronize()
    assert all(torch.equal(y, want) for y in got)
    small.close()
    for s in streams:
        assert hip.hipStreamDestroy(s) == 0


@pytest.mark.parametrize("first", ["nothing", "call", "call on another stream", "graph", "solve"])
@pytest.mark.parametrize("precond", [hb.PRECOND_NONE, hb.PRECOND_JACOBI])
def test_unallocated_solve_after_other_users(first, precond):
    """hb_cg_solve_noalloc finds a halo, without an allocation, whoever used the mesh before,
    and beside another thread's calls."""
    say(f"[case] no-allocation solve after {first}, precond={precond}")
    kw = dict(max_iter=30, precond=precond)
    ref = hb.Mesh(9, 8, 7, 5, jitter=0.1, seed=6)
    x = torch.as_tensor(inputs.random_vector(ref.NG, 96), device=DEV)
    ref.cg(1.3, x, want := torch.empty_like(x), **kw)
    y = ref.ax(1.3, x, torch.empty_like(x))
    m = hb.Mesh(9, 8, 7, 5, jitter=0.1, seed=6)
    other = torch.cuda.Stream()
    torch.cuda.synchronize()
    if first == "call":
        m.ax(1.3, x, torch.empty_like(x))
    elif first == "call on another stream":
        m.ax(1.3, x, torch.empty_like(x), stream=other)
    elif first == "graph":
        g = torch.cuda.CUDAGraph()
        captured = torch.empty_like(x)
        with torch.cuda.graph(g, stream=other):
            m.ax(1.3, x, captured)
    elif first == "solve":
        m.cg(1.3, x, torch.empty_like(x), **kw)
    held = m.device_bytes()
    m.cg_noalloc(1.3, x, got := torch.empty_like(x), **kw)
    assert m.device_bytes() == held
    assert torch.equal(got, want)
    ys, stream = out_like(x, 100), torch.cuda.current_stream()

    def work():
        for v in ys:
            m.ax(1.3, x, v, stream=stream)

    t = threading.Thread(target=work)
    t.start()
    sols = out_like(x, 3)
    for s in sols:
        m.cg_noalloc(1.3, x, s, stream=stream, **kw)
    t.join()
    if first == "graph":
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(captured, y)
    torch.cuda.synchronize()
    assert all(torch.equal(s, want) for s in sols) and all(torch.equal(v, y) for v in ys)
    m.close()
    ref.close()
