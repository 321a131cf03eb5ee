"""Tiles whose DOFs lie 4 GiB or more apart: the operator forms 64-bit offsets there.
Such a box is too large for the oracle, but with the other workgroup shape its tiles are
not wide, so the two shapes check each other (1e-12, and 2e-5 for the FP32 operator, the
bounds of the other operator tests)."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2202_12477_amd as hb  # noqa: E402

DEV = torch.device("cuda:0")


def relerr(a, b):
    return float(torch.linalg.vector_norm(a - b) / torch.linalg.vector_norm(b))


# 780 and 900 million DOFs; test_plan.py checks that these boxes are wide in one shape only
@pytest.mark.parametrize("nx,ny,nz,N,dirichlet", [(1, 5_000_000, 4, 3, False), (1, 1_650_000, 2, 7, True)])
def test_wide_tiles_against_narrow_ones(nx, ny, nz, N, dirichlet):
    print(f"[case] wide tiles {nx}x{ny}x{nz} N={N} dirichlet={dirichlet}", flush=True)
    if torch.cuda.mem_get_info()[0] < 64 << 30:
        pytest.skip("needs 64 GiB of device memory")
    precs = (hb.PREC_FP64, hb.PREC_FP32_RR)
    saved = {p: hb.get_schedule(N, p) for p in precs}
    m = hb.Mesh(nx, ny, nz, N, jitter=0.1, seed=N, fp32=True, dirichlet=dirichlet)
    x = hb.rhs_uniform(torch.empty(m.NG, dtype=torch.float64, device=DEV), 5)
    y, y32 = [], []
    try:
        for v in (0, 2):
            for p in precs:
                hb.set_schedule(N, p, v)
            y.append(m.ax(1.3, x, torch.full_like(x, float("nan"))))
            y32.append(m.ax_f32(1.3, x, torch.full((m.NG,), float("nan"), dtype=torch.float32, device=DEV)))
        torch.cuda.synchronize()
    finally:
        for p, v in saved.items():
            hb.set_schedule(N, p, v)
    assert relerr(y[0], y[1]) <= 1e-12
    for z in y32:
        assert relerr(z.double(), y[1]) <= 2e-5
    m.close()
    del x, y, y32
    torch.cuda.empty_cache()
