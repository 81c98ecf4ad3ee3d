"""The fused network where a workgroup takes several tiles in turn, at each tile height: the weights
that it stages for its next tile beside the last layer's products must be in place when the next tile
reads them, also those staged by waves that have no products in the last layer (at 6, 10 and 12 rows)."""
import numpy as np
import pytest

from tests import test_gpu_cnn

pytestmark = pytest.mark.gpu


# rows per tile, rounds of the 256 workgroups: 6 x 4, 10 x 2, 10 x 5, 12 x 3, 12 x 7, 16 x 4
@pytest.mark.parametrize("shape", [(5, 30001), (229, 622), (454, 851), (347, 781), (1180, 554), (375, 1265)])
def test_several_tiles_per_workgroup_equal_the_chain(shape):
    for seed in range(3):
        test_gpu_cnn.test_fused_network_equals_the_layer_by_layer_chain(np.random.Generator(np.random.PCG64(seed)), shape)
