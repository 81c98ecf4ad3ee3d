"""The row pipelines of the model variants: streamed passes of 1 to 4 steps at several band heights give
the state of the register tiles bit for bit, the same maxima, the volumes up to the order of their sums."""
import pytest

from paper_1711_04471_amd.sw2d import Sw2d
from tests.test_gpu_block import _same, _variant_case

pytestmark = pytest.mark.gpu

CALLS = [9, 1, 3]


def _run(case, flags, streaming, spp=1, rows=None):
    with Sw2d.from_case(case, flags=flags, cd=0.5, hmin=0.0625) as sim:
        sim.streaming = streaming
        if rows:
            sim.band_rows = rows
        if spp > 1:
            sim.set_time_blocking(spp, rows=rows)
        assert sim.streaming == streaming
        for n in CALLS:
            sim.step(n)
        return sim.state_numpy(), sim.reduce(sum(CALLS))


@pytest.mark.parametrize("flags", [1, 2, 3, 8])
@pytest.mark.parametrize("shape", [(130, 257), (301, 97), (61, 200)])
def test_streamed_k_steps_of_a_variant_equal_tiles(shape, flags):
    c = _variant_case(shape, flags)
    want = _run(c, flags, False)
    for spp in (2, 3, 4):
        for rows in (8, 40):
            _same(_run(c, flags, True, spp, rows), want, c)


@pytest.mark.parametrize("flags", range(9))
@pytest.mark.parametrize("shape", [(200, 173), (131, 41)])
def test_streamed_band_heights_equal_tiles(shape, flags):
    c = _variant_case(shape, flags)
    want = _run(c, flags, False)
    for rows in (8, 16, 40, shape[1]):
        _same(_run(c, flags, True, 1, rows), want, c)
