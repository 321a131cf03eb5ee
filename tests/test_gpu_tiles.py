"""The assembled operator's tiles and the CG steps at the sizes where their forms
change, against the oracle:
  - boxes of several tiles in every direction with short last tiles, for every degree,
    plain and Dirichlet, both mass kinds, both shapes of workgroup: y = A x and
    y += A x to 1e-12 and the FP32 operator to 2e-5 (the bounds of the other operator
    tests), and twice the same bits;
  - CG around the single-workgroup tail of an iteration (up to 4096 DOFs), around a
    chunk of 1024 DOFs, and around the 2048 partial sums up to which alpha and beta are
    formed in the vector kernels: the first residual norms against the oracle's.  Both
    run the same recurrence on data that agree to about 1e-15 and a few steps amplify
    rounding by far less than 1e4: 1e-10."""
import sys

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
    return t.cpu().numpy()


def relerr(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.fixture(autouse=True)
def restore_table():
    saved = {(N, p): hb.get_schedule(N, p) for N in range(1, 16) for p in (hb.PREC_FP64, hb.PREC_FP32_RR)}
    yield
    for (N, p), v in saved.items():
        hb.set_schedule(N, p, v)


BOXES = [(19, 9, 7, 1), (17, 7, 5, 2), (13, 7, 5, 3), (11, 5, 3, 4), (15, 3, 2, 5), (11, 2, 3, 6), (9, 3, 3, 7),
         (7, 2, 2, 8), (5, 3, 2, 9), (2, 5, 2, 10), (3, 2, 2, 11), (2, 2, 3, 12), (2, 3, 2, 13), (3, 2, 2, 14),
         (2, 2, 2, 15)]


@pytest.mark.parametrize("nx,ny,nz,N", BOXES)
@pytest.mark.parametrize("dirichlet,mass", [(False, hb.MASS_GWJ), (False, hb.MASS_INVDEG), (True, hb.MASS_GWJ),
                                            (True, hb.MASS_INVDEG)])
def test_operator_over_several_tiles(nx, ny, nz, N, dirichlet, mass):
    say(f"[case] {nx}x{ny}x{nz} N={N} dirichlet={dirichlet} mass={mass}")
    m = hb.Mesh(nx, ny, nz, N, jitter=0.1, seed=N, fp32=True, dirichlet=dirichlet, mass=mass)
    ref = oracle.Mesh(nx, ny, nz, N, jitter=0.1, seed=N, dirichlet=dirichlet, mass=mass)
    x = inputs.random_vector(m.NG, 70 + N)
    yr = ref.ax(x, 1.3)
    xd = torch.as_tensor(x, device=DEV)
    for v in [0, 2] if N <= 7 else [0]:
        hb.set_schedule(N, hb.PREC_FP64, v)
        hb.set_schedule(N, hb.PREC_FP32_RR, v)
        y = torch.full_like(xd, float("nan"))  # overwritten, never read
        m.ax(1.3, xd, y)
        assert relerr(host(y), yr) <= 1e-12
        again = torch.empty_like(xd)
        m.ax(1.3, xd, again)
        assert torch.equal(y, again)
        m.ax_add(1.3, xd, y)
        assert relerr(host(y), 2.0 * yr) <= 1e-12
        y32 = torch.full((m.NG,), float("nan"), dtype=torch.float32, device=DEV)
        m.ax_f32(1.3, xd, y32)
        assert relerr(host(y32).astype(np.float64), yr) <= 2e-5
    m.close()


# NG = 4096, 4352; 1000, 1024, 1089; 2000 and 2084 chunks of DOFs; 1980 and 2197 tiles
STEPS = [(15, 15, 15, 1), (16, 15, 15, 1), (9, 9, 9, 1), (15, 7, 7, 1), (10, 10, 8, 1), (18, 18, 18, 7),
         (19, 18, 18, 7), (11, 12, 15, 11), (13, 13, 13, 11)]


@pytest.mark.parametrize("nx,ny,nz,N", STEPS)
@pytest.mark.parametrize("jacobi", [False, True])
def test_cg_steps_at_the_edges_of_their_forms(nx, ny, nz, N, jacobi):
    m = hb.Mesh(nx, ny, nz, N, jitter=0.05, seed=3)
    say(f"[case] CG steps {nx}x{ny}x{nz} N={N} NG={m.NG} jacobi={jacobi}")
    ref = oracle.Mesh(nx, ny, nz, N, jitter=0.05, seed=3)
    b = torch.empty(m.NG, dtype=torch.float64, device=DEV)
    hb.rhs_uniform(b, 5)
    x = torch.empty_like(b)
    its = 5
    res = m.cg(1.0, b, x, max_iter=its, fixed_iters=True, precond=hb.PRECOND_JACOBI if jacobi else hb.PRECOND_NONE)
    bh = oracle.rhs(m.NG, 5)
    hist = (ref.pcg if jacobi else ref.cg)(bh, 1.0, fixed_iters=its)["res"]
    got = np.asarray(res.history[: its + 1])
    err = np.max(np.abs(got - hist[: its + 1]) / np.abs(hist[: its + 1]))
    say(f"  history error {err:.2e}")
    assert err <= 1e-10
    m.close()


@pytest.mark.parametrize("schedule", [0, 2])
def test_persistent_launch_takes_its_own_tiles(schedule):
    """The persistent batched launch works in 256-thread tiles whatever shape the schedule
    table gives the per-step launches: same solution as the single solve (1e-9, as the
    other persistent tests)."""
    cases = [(4, 3), (3, 5), (3, 7), (2, 9)]
    ms, bs, xs = [], [], []
    for n, N in cases:
        if N <= 7:
            hb.set_schedule(N, hb.PREC_FP64, schedule)
        m = hb.Mesh(n, n, n, N, jitter=0.05, seed=N)
        b = torch.empty(m.NG, dtype=torch.float64, device=DEV)
        hb.rhs_uniform(b, 20 + N)
        ms.append(m)
        bs.append(b)
        xs.append(torch.full_like(b, float("nan")))
    st, res = hb.batch_solve(ms, [1.0] * len(ms), bs, xs, max_iter=40, fixed_iters=True, persistent=True)
    assert st == hb.HB_OK
    for (n, N), m, b, x, r in zip(cases, ms, bs, xs, res):
        say(f"[case] persistent {n}^3 N={N} schedule {schedule}")
        assert r.persistent_segments >= 1
        x1 = torch.empty_like(b)
        m.cg(1.0, b, x1, max_iter=40, fixed_iters=True)
        assert relerr(host(x), host(x1)) <= 1e-9


@pytest.mark.parametrize("dirichlet", [False, True])
@pytest.mark.parametrize("prec", [hb.PREC_FP64, hb.PREC_FP32_RR])
@pytest.mark.parametrize("schedule", [None, 2])
def test_operator_of_every_degree_in_one_launch(schedule, prec, dirichlet):
    """A batch of all degrees runs their operators in one launch, a batch of one problem
    in its degree's own: the same bits (the same sums in the same order); and the FP32
    operator's solves meet their tolerance by the FP64 operator."""
    ms, bs, xs = [], [], []
    for N in range(1, 16):
        if schedule is not None and N <= 7:
            hb.set_schedule(N, prec, schedule)
        n = {1: 12, 2: 7, 3: 5}.get(N, 3 if N < 10 else 2)
        m = hb.Mesh(n, n, n, N, jitter=0.05, seed=N, fp32=True, dirichlet=dirichlet)
        b = torch.empty(m.NG, dtype=torch.float64, device=DEV)
        hb.rhs_uniform(b, 40 + N)
        ms.append(m)
        bs.append(b)
        xs.append(torch.full_like(b, float("nan")))
    fixed = prec == hb.PREC_FP64
    st, res = hb.batch_solve(ms, [1.0] * 15, bs, xs, max_iter=8 if fixed else 5000, fixed_iters=fixed,
                             rtol=0.0 if fixed else 1e-6, prec=prec)
    assert st == hb.HB_OK
    for N, (m, b, x, r) in enumerate(zip(ms, bs, xs, res), 1):
        say(f"[case] any degree: N={N} prec={prec} dirichlet={dirichlet} schedule={schedule}")
        if fixed:
            x1 = torch.full_like(b, float("nan"))
            hb.batch_solve([m], [1.0], [b], [x1], max_iter=8, fixed_iters=True)
            assert torch.equal(x, x1)
        else:
            y = torch.empty_like(b)
            m.ax(1.0, x, y)
            assert relerr(host(y), host(b)) <= 1.2e-6


@pytest.mark.parametrize("nx,ny,nz,N", BOXES)
@pytest.mark.parametrize("dirichlet,mass", [(False, hb.MASS_GWJ), (True, hb.MASS_INVDEG)])
def test_jacobi_diagonal_of_every_degree(nx, ny, nz, N, dirichlet, mass):
    """The preconditioner's diagonal is formed from the elements' maps: the first residual
    norms of the preconditioned solve against the oracle's (1e-10, as above)."""
    say(f"[case] Jacobi {nx}x{ny}x{nz} N={N} dirichlet={dirichlet} mass={mass}")
    m = hb.Mesh(nx, ny, nz, N, jitter=0.1, seed=N, dirichlet=dirichlet, mass=mass)
    ref = oracle.Mesh(nx, ny, nz, N, jitter=0.1, seed=N, dirichlet=dirichlet, mass=mass)
    b = torch.empty(m.NG, dtype=torch.float64, device=DEV)
    hb.rhs_uniform(b, 6)
    x = torch.empty_like(b)
    res = m.cg(1.3, b, x, max_iter=4, fixed_iters=True, precond=hb.PRECOND_JACOBI)
    hist = ref.pcg(oracle.rhs(m.NG, 6), 1.3, fixed_iters=4)["res"]
    assert np.max(np.abs(np.asarray(res.history[:5]) - hist[:5]) / hist[:5]) <= 1e-10
    m.close()


@pytest.mark.parametrize("nx,ny,nz,N", [(5, 3, 2, 2), (129, 3, 2, 14), (33, 32, 9, 5)])
@pytest.mark.parametrize("dirichlet", [False, True])
def test_export_by_pieces(nx, ny, nz, N, dirichlet):
    """Z bit for bit and the factors to rounding (1e-13 of the largest of each), in one
    piece and in several (more than 2^21 nodes)."""
    say(f"[case] export {nx}x{ny}x{nz} N={N} dirichlet={dirichlet}")
    m = hb.Mesh(nx, ny, nz, N, jitter=0.1, seed=2, dirichlet=dirichlet, mass=hb.MASS_INVDEG)
    ref = oracle.Mesh(nx, ny, nz, N, jitter=0.1, seed=2, dirichlet=dirichlet, mass=hb.MASS_INVDEG)
    geo, mp, _, _, _ = m.export()
    assert np.array_equal(np.asarray(mp).ravel().astype(np.int64), ref.map)
    g, gr = np.asarray(geo).reshape(m.E, 7, -1), ref.geo.reshape(m.E, 7, -1).copy()
    gr[:, 6][ref.map.reshape(m.E, -1) < 0] = 0.0  # the library's mass of a node without a DOF; the oracle does not mask it
    for f in range(7):
        assert np.max(np.abs(g[:, f] - gr[:, f])) <= 1e-13 * np.max(np.abs(gr[:, f]))
    m.close()


# local nodes on both sides of the one-launch addition's line (3 * 2^19), and tiny boxes
ADDS = [(1, 1, 1, 3), (2, 1, 3, 7), (5, 4, 3, 5), (14, 14, 14, 7), (15, 14, 15, 7), (58, 58, 58, 1), (59, 58, 58, 1),
        (11, 11, 11, 9), (12, 12, 11, 9), (7, 7, 7, 15), (8, 7, 7, 15)]


@pytest.mark.parametrize("nx,ny,nz,N", ADDS)
@pytest.mark.parametrize("dirichlet,gather", [(False, False), (True, False), (False, True), (True, True)])
def test_added_in_one_launch_or_two(nx, ny, nz, N, dirichlet, gather):
    """y += A x by either route against the oracle (1e-12); on a reproducible mesh the same
    bits every time."""
    say(f"[case] y += A x {nx}x{ny}x{nz} N={N} dirichlet={dirichlet} gather={gather}")
    m = hb.Mesh(nx, ny, nz, N, jitter=0.1, seed=N, dirichlet=dirichlet, gather=gather)
    ref = oracle.Mesh(nx, ny, nz, N, jitter=0.1, seed=N, dirichlet=dirichlet)
    x, y0 = inputs.random_vector(m.NG, 70 + N), inputs.random_vector(m.NG, 80 + N)
    want = y0 + ref.ax(x, 1.3)
    xd = torch.as_tensor(x, device=DEV)
    ys = [m.ax_add(1.3, xd, torch.as_tensor(y0, device=DEV).clone()) for _ in range(4)]
    assert max(relerr(host(y), want) for y in ys) <= 1e-12
    if gather:
        assert all(torch.equal(y, ys[0]) for y in ys)
    m.close()
