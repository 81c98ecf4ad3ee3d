"""SOR on long narrow columns, whose launches hold more workgroups than one launch dimension."""
import pytest
import torch

from paper_1711_04471_amd.sw2d import SorSolver
from tests.test_gpu_sor import RES_TOL, TOL

pytestmark = pytest.mark.gpu


def _solve(p, f, omega, iters):
    """Red-black sweeps in FP64 (unit spacings), on the device."""
    nz, ny, nx = p.shape
    z = torch.arange(1, nz - 1, device=p.device)
    for _ in range(iters):
        for colour in (0, 1):
            for j in range(1, ny - 1):
                for i in range(1, nx - 1):
                    nb = p[1:-1, j, i + 1] + p[1:-1, j, i - 1] + p[1:-1, j + 1, i] + p[1:-1, j - 1, i] + \
                        p[2:, j, i] + p[:-2, j, i]
                    old = p[1:-1, j, i]
                    new = old + omega * ((nb - f[1:-1, j, i]) / 6 - old)
                    p[1:-1, j, i] = torch.where((z + i + j) % 2 == colour, new, old)
    return p


# 17,000,000 planes of one workgroup each (the layout passes) and of 4 to a workgroup (70,000,000: the
# sweeps as well); below them a column that fits one dimension
@pytest.mark.parametrize("nx,nz", [(3, 400_001), (3, 17_000_001), (4, 70_000_002)])
def test_long_columns(nx, nz):
    ny, iters, omega = 3, 2, 1.5
    print(f"sor column {nx} x {ny} x {nz}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(nx)
    p = torch.randn(nz, ny, nx, device="cuda", generator=gen)
    f = torch.randn(nz, ny, nx, device="cuda", generator=gen)
    want = _solve(p.double(), f.double(), omega, iters)
    solver = SorSolver(nx, ny, nz, 1.0, 1.0, 1.0, omega, iters)
    solver.run(p, f)
    res = solver.residuals()
    assert (p.double() - want).norm() <= TOL * want.norm()
    q = want
    r = f.double()[1:-1, 1, 1:-1] - (q[1:-1, 1, 2:] + q[1:-1, 1, :-2] + q[1:-1, 0, 1:-1] + q[1:-1, 2, 1:-1] +
                                     q[2:, 1, 1:-1] + q[:-2, 1, 1:-1] - 6 * q[1:-1, 1, 1:-1])
    assert abs(res["sum_r2"][-1] / float((r * r).sum()) - 1) <= RES_TOL
    assert abs(res["max_abs_r"][-1] / float(r.abs().max()) - 1) <= RES_TOL
