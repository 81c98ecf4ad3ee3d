"""The grids that a persistent launch may be asked for, also larger ones than the device holds at once."""
import numpy as np
import pytest
import torch

from paper_1711_04471_amd import _lib, inputs
from paper_1711_04471_amd.sw2d import Sw2dBatch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,per_cu", [(1, 6), (2, 5), (3, 4)])
def test_grids_up_to_the_limit_are_taken(K, per_cu):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    # more tiles than any of the grids has workgroups
    cases = [inputs.small_basin(1500, 1301, seed=k) for k in range(2)] + [inputs.small_basin(129, 65, seed=9)]
    n, got = 6 * K, []
    for grid in (0, 100, 3 * cus + 1, per_cu * cus):
        with Sw2dBatch(cases, band_rows=[8] * 3) as b:
            b.set_time_blocking(K)
            b.set_launch(7, False, grid)
            assert b.grid == (grid or per_cu * cus)
            with pytest.raises(_lib.Sw2dError):
                b.set_launch(7, False, per_cu * cus + 1)
            b.step(n)
            red = b.reduce()  # (fails if a barrier waited in vain)
            got.append(([x for k in range(b.n) for x in b.state_numpy(k)], red))
    for states, red in got[1:]:
        # (a launch per pass takes other passes, whose tiles group the sums otherwise)
        assert np.array_equal(red, got[1][1])
        for x, y in zip(states, got[0][0]):
            assert np.array_equal(x, y)


def test_more_steps_per_pass_lower_the_grid():
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    with Sw2dBatch([inputs.small_basin(64, 64, seed=1)]) as b:
        b.set_time_blocking(3)
        assert b.grid == 4 * cus
        b.set_time_blocking(1)
        assert b.grid == 4 * cus
        b.set_launch(50, True, 0)
        assert b.grid == 6 * cus
