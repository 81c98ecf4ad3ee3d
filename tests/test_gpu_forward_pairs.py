"""The training forward (two layers per launch) equals the layer-by-layer convolutions bit for bit, at
the edges of its 16 x 32 tiles, over several tiles per workgroup, and on images too wide for them."""
import ctypes

import numpy as np
import pytest
import torch

from tests.test_gpu_cnn import DEV, bf16, check, lib, ptr, stream

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 16, 32), (1, 17, 33), (2, 15, 31), (3, 31, 65), (2, 300, 401),
                                   (1, 2, 840000)])
def test_training_forward_equals_the_layers(shape):
    N, H, W = shape
    rng = np.random.Generator(np.random.PCG64(H * W))
    x = torch.zeros((N, H, W, 16), dtype=torch.bfloat16, device=DEV)
    gen = torch.Generator(device=DEV).manual_seed(H)
    x[..., :5] = torch.randn((N, H, W, 5), generator=gen, device=DEV).to(torch.bfloat16)
    wk = [bf16(rng.standard_normal((9, 32, c)) * 0.1)[0] for c in (16, 32, 32, 32)]
    bias = [torch.from_numpy(rng.standard_normal(32).astype(np.float32)).to(DEV) for _ in range(4)]
    maps = lambda: [torch.full((N, H, W, 32), float("nan"), dtype=torch.bfloat16, device=DEV) for _ in range(3)]
    planes = lambda: torch.full((N, 3, H, W), float("nan"), dtype=torch.float32, device=DEV)
    want, want_out, got, got_out = maps(), planes(), maps(), planes()
    for layer in range(4):
        src, cin = (x, 16) if layer == 0 else (want[layer - 1], 32)
        dst = want[layer] if layer < 3 else want_out
        check(lib().sw2d_conv3x3_fwd(ptr(src), cin, ptr(wk[layer]), ptr(bias[layer]), int(layer < 3), ptr(dst), N, H, W,
                                     stream()))
    arr = lambda ts: (ctypes.c_void_p * len(ts))(*[t.data_ptr() for t in ts])
    check(lib().sw2d_cnn_forward_train(ptr(x), arr(wk), arr(bias), arr(got), ptr(got_out), N, H, W, stream()))
    for a, b in zip([*got, got_out], [*want, want_out]):
        assert torch.equal(a, b)
