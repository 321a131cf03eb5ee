"""Calls that meet: the schedule table set by one host thread while another works."""
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
