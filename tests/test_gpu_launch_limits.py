"""Grids of so many rows that passes of the library's choice would need more threads than a launch
holds: windows of the result against the same rows stepped as a basin of their own."""
import pytest
import torch

from paper_1711_04471_amd.sw2d import Sw2d, Sw2dBatch

pytestmark = pytest.mark.gpu

MODEL = dict(dx=100.0, dy=100.0, g=9.81, dt=2.0, eps=0.05)


class _Column:
    """A basin one water cell wide, made on the device."""

    def __init__(self, ny, eta=None):
        self.nx, self.ny = 3, ny
        for k, v in MODEL.items():
            setattr(self, k, v)
        self.H = torch.full((ny, 3), 20.0, device="cuda")
        self.mask = torch.zeros((ny, 3), dtype=torch.uint8, device="cuda")
        self.mask[1:-1, 1] = 1
        if eta is None:
            gen = torch.Generator(device="cuda").manual_seed(1)
            eta = 0.1 * torch.randn((ny, 3), device="cuda", generator=gen)
        self.eta = eta * self.mask
        self.u = torch.zeros_like(self.H)
        self.v = torch.zeros_like(self.H)


def _check_windows(case, state, steps):
    """The first, the middle and the last rows; a step reaches two rows."""
    rows, reach = 512, 3 * steps
    for a in (0, case.ny // 2, case.ny - rows):
        lo, hi = max(a - reach, 0), min(a + rows + reach, case.ny)
        part = _Column(hi - lo, case.eta[lo:hi].clone())
        with Sw2d.from_case(part) as sim:
            sim.step(steps)
            # rows that the cut has not reached
            b, e = (a - lo if lo > 0 else 0), (a + rows - lo if hi < case.ny else hi - lo)
            for name, x, y in zip("euv", state, sim.state()):
                assert torch.equal(x[lo + b:lo + e], y[b:e]), (a, name)


@pytest.mark.parametrize("steps", [3, 4])
def test_more_rows_than_a_launch_of_low_bands_holds(steps):
    case = _Column((1 << 27) + 1001)
    with Sw2d.from_case(case) as sim:
        sim.band_rows = 64
        sim.step(steps)
        _check_windows(case, sim.state(), steps)


@pytest.mark.parametrize("launch", [None, (50, True, 0), (50, False, 64)])
def test_more_tiles_than_a_launch_per_pass_holds(launch):
    """24-row tiles own 8 rows at 4 steps per pass."""
    cases, steps = [_Column(40), _Column((1 << 26) + 1001), _Column(70)], 5
    with Sw2dBatch(cases, band_rows=[8] * 3) as b:
        if launch:
            b.set_launch(*launch)
        b.step(steps)
        for k, case in enumerate(cases):
            if case.ny < 512:
                with Sw2d.from_case(case) as sim:
                    sim.step(steps)
                    for x, y in zip(b.state(k), sim.state()):
                        assert torch.equal(x, y), k
            else:
                _check_windows(case, b.state(k), steps)
        assert (b.reduce()["step"] == steps).all()
