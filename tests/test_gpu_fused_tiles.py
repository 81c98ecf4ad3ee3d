"""The fused network at images that take each of its tile heights (6, 10, 12 and 16 rows), with partial
last tiles, against the layer-by-layer chain."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(5, 3), (97, 129), (221, 300), (299, 301), (403, 400), (517, 530)])
def test_every_tile_height_equals_the_chain(shape):
    from tests import test_gpu_cnn
    test_gpu_cnn.test_fused_network_equals_the_layer_by_layer_chain(np.random.Generator(np.random.PCG64(7)), shape)
