"""Weight gradients over many pixels: a wave's chain of FP32 additions stays at 1024 pixels however many
tiles a workgroup takes."""
import pytest
import torch

from tests.test_gpu_cnn import DEV, check, lib, ptr, stream

pytestmark = pytest.mark.gpu

# Every product of an output is the same positive number, so that the additions of a chain all round
# the same way for long. 32 x 1024^2 pixels are 256 tiles for each of 256 workgroups. One rounding of at
# most 2^-24 of the running sum each: 16 products of a matrix instruction and 64 of them per chain, the
# chains of a workgroup's waves (at most 132 additions), 8 workgroups per slice, 32 slices.
N, H, W = 32, 1024, 1024
DEPTH = 16 + 64 + 132 + 8 + 32


def _expected(value):
    """Pixels whose tap lies inside the image, times the product."""
    rows = torch.tensor([H - 1, H, H - 1], dtype=torch.float64)
    cols = torch.tensor([W - 1, W, W - 1], dtype=torch.float64)
    return (N * value * rows[:, None] * cols[None, :]).reshape(9, 1, 1)


@pytest.mark.parametrize("cin,channels", [(16, 0), (32, 0), (32, 32), (32, 4)])
@pytest.mark.parametrize("a,b", [(253 / 128, 137 / 128), (255 / 128, 131 / 128)])
def test_chains_stay_short(cin, channels, a, b):
    """channels 0: the weight gradient alone, else both gradients with a dy of that many channels."""
    x = torch.full((N, H, W, cin), b, dtype=torch.bfloat16, device=DEV)
    dy = torch.full((N, H, W, channels or 32), a, dtype=torch.bfloat16, device=DEV)
    dW = torch.empty((9, 32, cin), dtype=torch.float32, device=DEV)
    db = torch.empty(32, dtype=torch.float32, device=DEV)
    need = lib().sw2d_wgrad_workspace_bytes(cin, N, H, W)
    work = torch.empty(need, dtype=torch.uint8, device=DEV)
    if channels:
        wd = torch.zeros((9, 32, 32), dtype=torch.bfloat16, device=DEV)
        dx = torch.empty_like(x)
        check(lib().sw2d_conv3x3_backward(ptr(x), ptr(dy), channels, ptr(wd), ptr(dx), N, H, W, ptr(dW), ptr(db),
                                          ptr(work), need, stream()))
    else:
        check(lib().sw2d_conv3x3_wgrad(ptr(x), cin, ptr(dy), N, H, W, ptr(dW), ptr(db), ptr(work), need, stream()))
    outputs = min(channels or 32, 32)
    err = (dW.double().cpu() / _expected(a * b) - 1).abs()[:, :outputs].max().item()
    print(f"cin {cin} channels {channels}: dW {err:.2e}, allowed {DEPTH * 2**-24:.2e}", flush=True)
    assert err <= DEPTH * 2.0**-24
    assert not dW[:, outputs:].any()
    # a bias adds a few bits per pixel: its sums are exact
    assert (db[:outputs].double().cpu() == N * H * W * a).all() or \
        ((db[:outputs].double().cpu() / (N * H * W * a) - 1).abs() <= DEPTH * 2.0**-24).all()
