"""SOR on both sides of the switch between one launch per iteration (both colours of a position, fewer
than 655,360 positions of a colour) and two sweeps per iteration (4 planes per thread, from there on)."""
import numpy as np
import pytest
import torch

from paper_1711_04471_amd.sw2d import SorSolver
from tests.test_gpu_sor import _check, _fma, _gpu, _random_case

pytestmark = pytest.mark.gpu

SWITCH = 655_360


def _positions(shape):
    nz, ny, nx = shape
    return (nx + 1) // 2 * (ny - 2) * (nz - 2)


# the sweeps: inner planes that leave 1, 2, 3 and 0 of the last 4, one to 3 planes alone, a narrow and a
# flat grid, odd and even widths, the switch itself; below it the launch per iteration
SWEEPS = [(35, 202, 201), (36, 200, 200), (37, 190, 199), (38, 190, 197), (3, 1312, 1001), (4, 700, 941), (5, 440, 1002),
          (50_000, 9, 4), (9, 3, 187_301), (42, 130, 255), (42, 130, 256)]
PAIRS = [(42, 128, 259), (41, 130, 256), (1300, 11, 112)]


@pytest.mark.parametrize("shape", SWEEPS + PAIRS)
def test_either_path_matches_oracle(shape):
    assert (_positions(shape) >= SWITCH) == (shape in SWEEPS)
    c = _random_case(shape, seed=sum(shape), omega=1.5, iters=4)
    print(f"sor {shape}", flush=True)
    p, res = _gpu(c)
    _check(c, p, res, c.iters)


@pytest.mark.parametrize("shape", [(37, 190, 199), (36, 200, 200), (5, 440, 1002), (42, 128, 259)])
def test_either_path_bitwise(shape):
    """Against the two-colour sweeps in FP32 with their fused multiply-adds, as defined."""
    nz, ny, nx = shape
    c = _random_case(shape, seed=7, omega=1.7, iters=2)
    cs = [1.0 / h**2 for h in (c.dx, c.dy, c.dz)]
    cx, cy, cz, inv, om = (np.float32(v) for v in (*cs, 1.0 / (2 * sum(cs)), c.omega))
    p, f = c.p0.copy(), c.f
    solver = SorSolver(nx, ny, nz, c.dx, c.dy, c.dz, c.omega, c.iters)
    gp = torch.from_numpy(p.copy()).cuda()
    solver.run(gp, torch.from_numpy(f).cuda())
    k, j, i = np.ogrid[:nz, :ny, :nx]
    inner = np.zeros(p.shape, dtype=bool)
    inner[1:-1, 1:-1, 1:-1] = True
    for _ in range(c.iters):
        for colour in (0, 1):
            sx, sy, sz = np.zeros_like(p), np.zeros_like(p), np.zeros_like(p)
            sx[:, :, 1:-1] = p[:, :, 2:] + p[:, :, :-2]
            sy[:, 1:-1] = p[:, 2:] + p[:, :-2]
            sz[1:-1] = p[2:] + p[:-2]
            g = (_fma(cz, sz, _fma(cy, sy, cx * sx)) - f) * inv
            p = np.where(inner & ((i + j + k) % 2 == colour), _fma(om, g - p, p), p)
    assert np.array_equal(gp.cpu().numpy(), p)
