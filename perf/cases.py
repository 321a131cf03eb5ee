"""Timing cases of the library's public entry points (paper_2202_12477_amd).

listed() names the cases, draw() makes more of the same ranges, prepare() builds what a caller has in hand
(meshes, vectors, an engine), run() is one pass through the public calls, work() the bytes and operations such a
pass cannot do without, and exact() the same results from plain torch in 64 bits.

The kinds of a case and the calls they stand for:
  ax       y = A x (Mesh.ax): the operator by itself, every degree, plain and Dirichlet boxes, both mass terms
  two      the same on a mesh built with gather=True (results reproducible from run to run)
  ax32     y = A_32 x (Mesh.ax_f32): the FP32 operator of the mixed-precision solvers
  cg       Mesh.cg with a fixed number of iterations (the benchmark's way), plain or Jacobi, launches or graphs
  rr       Mesh.cg to a tolerance with the FP32 operator and FP64 residual replacement
  batch    batch_solve over uneven boxes, a fixed number of iterations
  engine   requests submitted to a serving Engine and stepped until every one is done
"""
import math
import random

import numpy as np
import torch

import paper_2202_12477_amd as hb

LAMBDA = 1.0
JITTER = 0.05


def _box(kind, name, nx, ny, nz, N, **more):
    case = {"name": name, "kind": kind, "nx": nx, "ny": ny, "nz": nz, "N": N, "jitter": JITTER, "dirichlet": False,
            "invdeg": False}
    case.update(more)
    return case


def listed():
    return [
        # the small verification box: one operator call, bound by launch latency
        _box("ax", "ax_small", 4, 4, 4, 3),
        # low degree on a ragged masked box (tiles straddle rows, the identity mass of the method's own equation)
        _box("ax", "ax_low_ragged", 61, 83, 47, 2, dirichlet=True, invdeg=True),
        # the benchmark's operator: 32^3 affine elements, N = 7
        _box("ax", "ax_main", 32, 32, 32, 7, jitter=0.0),
        # the top of the order sweep
        _box("ax", "ax_high", 16, 16, 16, 15),
        # FP32 operator at a degree whose elements do not fill whole waves
        _box("ax32", "ax_f32", 26, 26, 26, 9),
        # the reproducible operator at an ordinary size, ragged
        _box("two", "two_phase", 31, 30, 28, 5),
        # the small verification box: 100 iterations, bound by launch latency
        _box("cg", "cg_small", 4, 4, 4, 3, iters=100, jacobi=False, graph_k=0),
        # the benchmark itself: 100 iterations on the 32^3 box
        _box("cg", "cg_main", 32, 32, 32, 7, jitter=0.0, iters=100, jacobi=False, graph_k=0),
        # the largest single-device box of the method's own runs (50^3, N = 7, Dirichlet), deformed, Jacobi
        _box("cg", "pcg_large", 50, 50, 50, 7, dirichlet=True, iters=100, jacobi=True, graph_k=0),
        # a mixed-precision solve to a tight tolerance at a high degree
        _box("rr", "rr_solve", 11, 10, 9, 11, rtol=1e-11, jacobi=False),
        # uneven independent problems advanced together
        {"name": "batch", "kind": "batch", "count": 16, "low": 3, "high": 16, "iters": 50, "jacobi": False, "mix": 4},
        # a burst of served requests, each solved to its tolerance and copied back to the host
        {"name": "engine", "kind": "engine", "count": 16, "low": 8, "high": 512, "rtol": 1e-11, "jacobi": True,
         "mix": 5},
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _sides(rng, N, nodes):
    """Sides of a box of about `nodes` local nodes at degree N, of uneven proportions."""
    e = max(1.0, nodes / (N + 1) ** 3)
    cube = e ** (1.0 / 3.0)
    nx = max(1, round(cube * _log_uniform(rng, 0.6, 1.7)))
    ny = max(1, round(cube * _log_uniform(rng, 0.6, 1.7)))
    return nx, ny, max(1, round(e / (nx * ny)))


def draw(rng: random.Random):
    kind = rng.choice(["ax", "ax", "ax32", "two", "cg", "cg", "rr", "batch", "engine"])
    if kind == "batch":
        return {"kind": kind, "count": rng.randint(3, 40), "low": 3, "high": rng.randint(6, 18),
                "iters": rng.randint(20, 50), "jacobi": rng.random() < 0.5, "mix": rng.randrange(1 << 20)}
    if kind == "engine":
        return {"kind": kind, "count": rng.randint(2, 24), "low": 8, "high": round(_log_uniform(rng, 32, 1024)),
                "rtol": 1e-11, "jacobi": rng.random() < 0.5, "mix": rng.randrange(1 << 20)}
    N = rng.randint(1, 15)
    dirichlet = rng.random() < 0.35
    if kind == "rr":
        nx, ny, nz = _sides(rng, N, _log_uniform(rng, 2 ** 12, 2 ** 21))
    elif kind == "cg":
        nodes = _log_uniform(rng, 2 ** 9, 2 ** 24)
        nx, ny, nz = _sides(rng, N, nodes)
    else:
        nx, ny, nz = _sides(rng, N, _log_uniform(rng, 2 ** 9, 2 ** 24.5))
    if dirichlet:  # a masked box needs an interior node along every side
        nx, ny, nz = (max(n, 2) if N == 1 else n for n in (nx, ny, nz))
    case = _box(kind, "", nx, ny, nz, N, jitter=rng.choice([0.0, JITTER, 0.2]), dirichlet=dirichlet,
                invdeg=rng.random() < 0.2)
    del case["name"]
    if kind == "cg":
        # short runs on small systems, which CG solves in few iterations
        case.update(iters=rng.randint(10, 100 if nodes > 2 ** 16 else 40), jacobi=rng.random() < 0.4, graph_k=rng.choice([0, 0, 10]))
    elif kind == "rr":
        case.update(rtol=1e-11, jacobi=rng.random() < 0.5, jitter=JITTER, invdeg=False)
    return case


def _mixed_boxes(case):
    """The boxes of a batch or of a burst of requests: (nx, ny, nz, N) each, as the case's own stream gives them."""
    rng = random.Random(case["mix"])
    boxes = []
    for _ in range(case["count"]):
        if case["kind"] == "batch":  # cubic grids, four degrees
            n = rng.randint(case["low"], case["high"])
            boxes.append((n, n, n, rng.choice([3, 5, 7, 9])))
        else:  # near-cubic boxes of log-uniform element counts, five degrees
            e = _log_uniform(rng, case["low"], case["high"])
            nz = max(1, int(e ** (1.0 / 3.0)))
            ny = max(1, int(math.sqrt(e / nz)))
            boxes.append((max(1, round(e / (ny * nz))), ny, nz, rng.choice([3, 5, 7, 9, 11])))
    return boxes


def _global_nodes(nx, ny, nz, N, dirichlet=False):
    k = -1 if dirichlet else 1
    return (nx * N + k) * (ny * N + k) * (nz * N + k)


def _vector(n, seed, uniform):
    g = torch.Generator(device="cuda").manual_seed(seed)
    if uniform:  # the benchmark's forcing is uniform in [-1, 1)
        return torch.rand(n, generator=g, device="cuda", dtype=torch.float64) * 2.0 - 1.0
    return torch.randn(n, generator=g, device="cuda", dtype=torch.float64)


def _mesh(case, seed):
    return hb.Mesh(case["nx"], case["ny"], case["nz"], case["N"], jitter=case["jitter"], seed=seed,
                   mass=hb.MASS_INVDEG if case["invdeg"] else hb.MASS_GWJ, fp32=case["kind"] in ("ax32", "rr"),
                   dirichlet=case["dirichlet"], gather=case["kind"] == "two")


def prepare(case, seed):
    kind = case["kind"]
    if kind == "engine":
        # Mesh and forcing are made from seeds at admission, inside the engine
        engine = hb.Engine(8 << 30, 32, prec=hb.PREC_FP64, iters_per_step=25,
                           precond=hb.PRECOND_JACOBI if case["jacobi"] else hb.PRECOND_NONE)
        return {"case": case, "engine": engine, "seed": seed, "boxes": _mixed_boxes(case)}
    if kind == "batch":
        meshes, bs = [], []
        for i, (nx, ny, nz, N) in enumerate(_mixed_boxes(case)):
            meshes.append(hb.Mesh(nx, ny, nz, N, jitter=JITTER, seed=seed + i))
            bs.append(_vector(meshes[-1].NG, seed + i, True))
        return {"case": case, "meshes": meshes, "b": bs, "x": [torch.empty_like(b) for b in bs]}
    m = _mesh(case, seed)
    state = {"case": case, "mesh": m, "x": _vector(m.NG, seed, kind in ("cg", "rr"))}
    state["y"] = torch.empty(m.NG, device="cuda", dtype=torch.float32 if kind == "ax32" else torch.float64)
    return state


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "engine":
        e = state["engine"]
        seed = state["seed"]
        tickets = [e.submit(nx, ny, nz, N, jitter=JITTER, seed=seed + i, lam=LAMBDA, rhs_seed=seed + 1000 + i,
                            rtol=case["rtol"]) for i, (nx, ny, nz, N) in enumerate(state["boxes"])]
        while True:
            info = e.step()
            if not info["running"] and not info["queued"]:
                break
        return np.concatenate([e.poll(t)[1] for t in tickets])
    if kind == "batch":
        hb.batch_solve(state["meshes"], [LAMBDA] * len(state["meshes"]), state["b"], state["x"],
                       max_iter=case["iters"], fixed_iters=True,
                       precond=hb.PRECOND_JACOBI if case["jacobi"] else hb.PRECOND_NONE)
        return state["x"]
    m, x, y = state["mesh"], state["x"], state["y"]
    if kind in ("ax", "two"):
        return m.ax(LAMBDA, x, y)
    if kind == "ax32":
        return m.ax_f32(LAMBDA, x, y)
    precond = hb.PRECOND_JACOBI if case["jacobi"] else hb.PRECOND_NONE
    if kind == "cg":
        res = m.cg(LAMBDA, x, y, max_iter=case["iters"], fixed_iters=True, precond=precond, graph_k=case["graph_k"])
        return {"x": y, "history": np.array(res.history)}
    m.cg(LAMBDA, x, y, max_iter=100000, fixed_iters=False, rtol=case["rtol"], history=False, prec=hb.PREC_FP32_RR,
         precond=precond)
    return y


# Work.  The operator's inputs are the assembled vector and the box's vertices (everything else about the mesh
# follows from them), its output the assembled vector; its operations are the six contractions of (N+1)^4
# multiply-adds and the pointwise terms per element, as the method counts them.


def _ax_work(nx, ny, nz, N, ng, out_bytes=8):
    E = nx * ny * nz
    vertices = 24 * (nx + 1) * (ny + 1) * (nz + 1)
    return (8 + out_bytes) * ng + vertices, E * (12 * (N + 1) ** 4 + 18 * (N + 1) ** 3)


def _cg_work(nx, ny, nz, N, ng, iters, jacobi):
    """Per iteration the operator, r -= alpha Ap with its norm, and x += alpha p with p = r + beta p; b is read once."""
    ab, af = _ax_work(nx, ny, nz, N, ng)
    return iters * (ab + (64 + (16 if jacobi else 0)) * ng) + 8 * ng, iters * (af + 10 * ng)


def _iterations(nx, ny, nz, N, rtol):
    """About how many iterations such a solve takes: CG's count grows as the largest side over the smallest spacing."""
    return max(20, int(0.55 * max(nx, ny, nz) * N ** 1.4 * -math.log10(rtol)))


def work(case):
    kind = case["kind"]
    if kind in ("batch", "engine"):
        total = [0.0, 0.0]
        for nx, ny, nz, N in _mixed_boxes(case):
            it = case["iters"] if kind == "batch" else _iterations(nx, ny, nz, N, case["rtol"])
            b, f = _cg_work(nx, ny, nz, N, _global_nodes(nx, ny, nz, N), it, case["jacobi"])
            total = [total[0] + b, total[1] + f]
        return {"bytes": total[0], "flops": total[1]}
    box = case["nx"], case["ny"], case["nz"], case["N"]
    ng = _global_nodes(*box, case["dirichlet"])
    if kind == "cg":
        b, f = _cg_work(*box, ng, case["iters"], case["jacobi"])
    elif kind == "rr":
        b, f = _cg_work(*box, ng, _iterations(*box, case["rtol"]), case["jacobi"])
    else:
        b, f = _ax_work(*box, ng, 4 if kind == "ax32" else 8)
    return {"bytes": float(b), "flops": float(f)}


# The same results in plain torch, 64 bits.


def _gll(N):
    """Gauss-Lobatto-Legendre nodes and weights and the derivative matrix D[i][j] = l_j'(xi_i)."""
    P = np.polynomial.legendre.Legendre.basis(N)
    inner = np.polynomial.legendre.Legendre.basis(N).deriv().roots().real if N > 1 else np.empty(0)
    dP, ddP = P.deriv(), P.deriv(2)
    for _ in range(4):  # Newton steps on P_N'
        inner = inner - dP(inner) / ddP(inner)
    xi = np.concatenate([[-1.0], np.sort(inner), [1.0]])
    xi = 0.5 * (xi - xi[::-1])
    L = P(xi)
    w = 2.0 / (N * (N + 1) * L * L)
    D = np.zeros((N + 1, N + 1))
    for i in range(N + 1):
        for j in range(N + 1):
            if i != j:
                D[i, j] = L[i] / L[j] / (xi[i] - xi[j])
    D[0, 0], D[N, N] = -N * (N + 1) / 4.0, N * (N + 1) / 4.0
    return xi, w, D


def _splitmix(seed, stream, index):
    """Uniform [0, 1) numbers of splitmix64 stream `stream` of `seed` at the positions `index`."""
    gamma = np.uint64(0x9E3779B97F4A7C15)

    def mix(state, i):
        z = state + (i + np.uint64(1)) * gamma
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        return z ^ (z >> np.uint64(31))

    with np.errstate(over="ignore"):
        start = mix(np.array([seed], dtype=np.uint64), np.array([stream], dtype=np.uint64))
        return (mix(start, index.astype(np.uint64)) >> np.uint64(11)).astype(np.float64) * 2.0 ** -53


class _Exact:
    """The assembled operator A = S + lambda M (or lambda I) of a box, in plain torch."""

    def __init__(self, nx, ny, nz, N, jitter, seed, dirichlet=False, invdeg=False):
        n1, dev = N + 1, "cuda" if torch.cuda.is_available() else "cpu"
        self.n1, self.E, self.dev = n1, nx * ny * nz, dev
        xi, w, D = _gll(N)
        self.D = torch.tensor(D, device=dev)
        i, j, k = np.meshgrid(np.arange(nx + 1), np.arange(ny + 1), np.arange(nz + 1), indexing="ij")
        index = i + (nx + 1) * (j + (ny + 1) * k)
        inside = (i > 0) & (i < nx) & (j > 0) & (j < ny) & (k > 0) & (k < nz)
        V = np.stack([i / nx, j / ny, k / nz]).astype(np.float64)
        if jitter:
            for d, n in enumerate((nx, ny, nz)):
                V[d] += np.where(inside, jitter / n * (2.0 * _splitmix(seed, d + 1, index) - 1.0), 0.0)
        V = torch.tensor(V, device=dev)  # [3, nx+1, ny+1, nz+1]
        r = torch.tensor(xi, device=dev)
        lin = torch.stack([0.5 * (1.0 - r), 0.5 * (1.0 + r)])  # [corner, node]
        slope = torch.stack([torch.full_like(r, -0.5), torch.full_like(r, 0.5)])

        def corners(dx, dy, dz):  # [E, 3], elements x fastest
            c = V[:, dx:nx + dx, dy:ny + dy, dz:nz + dz]
            return c.permute(3, 2, 1, 0).reshape(-1, 3)

        jac = []  # jac[d] = d x / d r_d, each [3][E, c, b, a]
        for d in range(3):
            f = [slope if d == q else lin for q in range(3)]
            J = torch.zeros(3, self.E, n1, n1, n1, device=dev, dtype=torch.float64)
            for dx in (0, 1):
                for dy in (0, 1):
                    for dz in (0, 1):
                        shape = f[2][dz][:, None, None] * f[1][dy][None, :, None] * f[0][dx][None, None, :]
                        X = corners(dx, dy, dz)
                        for q in range(3):
                            J[q] += X[:, q, None, None, None] * shape
            jac.append(J)

        def cross(u, v):
            return [u[1] * v[2] - u[2] * v[1], u[2] * v[0] - u[0] * v[2], u[0] * v[1] - u[1] * v[0]]

        cof = [cross(jac[1], jac[2]), cross(jac[2], jac[0]), cross(jac[0], jac[1])]
        det = sum(jac[0][q] * cof[0][q] for q in range(3))
        del jac
        W = torch.tensor(w, device=dev)
        www = W[:, None, None] * W[None, :, None] * W[None, None, :]
        s = www / det
        self.G = {(p, q): s * sum(cof[p][m] * cof[q][m] for m in range(3)) for p in range(3) for q in range(p, 3)}
        del cof
        # global numbers, -1 where a masked box has no unknown
        gx, gy, gz = nx * N + 1, ny * N + 1, nz * N + 1
        at = [torch.arange(n, device=dev)[:, None] * N + torch.arange(n1, device=dev)[None, :] for n in (nx, ny, nz)]
        I = at[0][None, None, :, None, None, :]
        J = at[1][None, :, None, None, :, None]
        K = at[2][:, None, None, :, None, None]
        shape = (nz, ny, nx, n1, n1, n1)
        if dirichlet:
            g = (I - 1) + (gx - 2) * ((J - 1) + (gy - 2) * (K - 1))
            on = (I > 0) & (I < gx - 1) & (J > 0) & (J < gy - 1) & (K > 0) & (K < gz - 1)
            self.ng = (gx - 2) * (gy - 2) * (gz - 2)
            g = torch.where(on, g, torch.full_like(g, self.ng))
        else:
            self.ng = gx * gy * gz
            g = I + gx * (J + gy * K)
        self.map = g.expand(shape).reshape(-1)
        self.on = torch.nonzero(self.map < self.ng).flatten() if dirichlet else None
        if invdeg:
            count = self.assemble(torch.ones_like(self.map, dtype=torch.float64))
            self.mass = torch.cat([1.0 / count, count.new_zeros(1)])[self.map].view_as(det)
        else:
            self.mass = www * det

    def _along(self, M, u, d):
        """M applied along direction d (0: r, 1: s, 2: t) of u [E, c, b, a]."""
        n1 = self.n1
        if d == 0:
            return (u.reshape(-1, n1) @ M.T).view_as(u)
        v = u.transpose(3 - d, 3).contiguous()
        return (v.reshape(-1, n1) @ M.T).view_as(v).transpose(3 - d, 3)

    def assemble(self, u):
        y = torch.zeros(self.ng, device=self.dev, dtype=torch.float64)
        u = u.reshape(-1)
        return y.index_add_(0, self.map, u) if self.on is None else y.index_add_(0, self.map[self.on], u[self.on])

    def ax(self, x):
        n1 = self.n1
        q = torch.cat([x, x.new_zeros(1)])[self.map].view(self.E, n1, n1, n1)
        dq = [self._along(self.D, q, d) for d in range(3)]
        u = LAMBDA * self.mass * q
        for d in range(3):
            f = sum(self.G[min(d, e), max(d, e)] * dq[e] for e in range(3))
            u += self._along(self.D.T, f, d)
        return self.assemble(u)

    def inverse_diagonal(self):
        D = self.D
        u = LAMBDA * self.mass
        for d in range(3):
            u = u + self._along((D * D).T, self.G[d, d], d)
        c = torch.diagonal(D)
        along = [c[None, None, None, :], c[None, None, :, None], c[None, :, None, None]]
        for p, q in ((0, 1), (0, 2), (1, 2)):
            u = u + 2.0 * along[p] * along[q] * self.G[p, q]
        return 1.0 / self.assemble(u)

    def cg(self, b, iters, rtol, jacobi):
        """Conjugate gradients from zero: (x, residual norms)."""
        inv = self.inverse_diagonal() if jacobi else None
        x, r = torch.zeros_like(b), b.clone()
        z = r * inv if jacobi else r
        p = z.clone()
        rho, history = torch.dot(r, z), [torch.linalg.vector_norm(r)]
        stop = rtol * float(history[0])
        for j in range(iters):
            Ap = self.ax(p)
            alpha = rho / torch.dot(p, Ap)
            x += alpha * p
            r -= alpha * Ap
            history.append(torch.linalg.vector_norm(r))
            if stop and float(history[-1]) <= stop:
                break
            z = r * inv if jacobi else r
            rho, old = torch.dot(r, z), rho
            p = z + (rho / old) * p
        return x, torch.stack(history)


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        out = []
        for i, (nx, ny, nz, N) in enumerate(_mixed_boxes(case)):
            A = _Exact(nx, ny, nz, N, JITTER, seed + i)
            out.append(A.cg(_vector(A.ng, seed + i, True), case["iters"], 0.0, case["jacobi"])[0])
        return out
    if kind == "engine":
        if sum((N + 1) ** 3 * nx * ny * nz for nx, ny, nz, N in _mixed_boxes(case)) > 2 ** 22:
            return None
        out = []
        for i, (nx, ny, nz, N) in enumerate(_mixed_boxes(case)):
            A = _Exact(nx, ny, nz, N, JITTER, seed + i)
            b = torch.tensor(2.0 * _splitmix(seed + 1000 + i, 0, np.arange(A.ng)) - 1.0, device=A.dev)
            out.append(A.cg(b, 20000, 0.01 * case["rtol"], True)[0])
        return torch.cat(out).cpu().numpy()
    A = _Exact(case["nx"], case["ny"], case["nz"], case["N"], case["jitter"], seed, case["dirichlet"], case["invdeg"])
    x = _vector(A.ng, seed, kind in ("cg", "rr"))
    if kind in ("ax", "two", "ax32"):
        return A.ax(x)
    if kind == "cg":
        y, history = A.cg(x, case["iters"], 0.0, case["jacobi"])
        return {"x": y, "history": history.cpu().numpy()}
    if A.ng * _iterations(case["nx"], case["ny"], case["nz"], case["N"], case["rtol"]) > 1e10:
        return None
    return A.cg(x, 20000, 0.01 * case["rtol"], True)[0]
