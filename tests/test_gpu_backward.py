"""The backward kernel (both gradients of a layer in one pass) against the separate data gradient
(bitwise) and the FP64 oracle, at the edges of its 16 x 32 tiles and workspaces."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import cnn_ref
from paper_1711_04471_amd import _lib
from tests.test_gpu_cnn import DEV, bf16, check, lib, ptr, stream

pytestmark = pytest.mark.gpu

# a weight sums one product per pixel in FP32: in chains of at most 16 products x 8 rows x 2 blocks
# per tile and at most 4 tiles here, then 8 waves, 8 workgroups per slice and 32 slices
DEPTH = 16 * 8 * 2 * 4 + 8 + 8 + 32
SHAPES = [(1, 1, 1), (1, 16, 32), (2, 17, 33), (1, 15, 31), (3, 40, 70), (1, 130, 200)]


def _oracle(x, dy):
    """dW [9][32][cin] and db in FP64, and the sums of the products' magnitudes."""
    out = []
    for a, d in ((x, dy), (np.abs(x), np.abs(dy))):
        w, b = 0.0, 0.0
        for n in range(len(a)):
            gw, gb = cnn_ref.conv3x3_wgrad(np.transpose(a[n], (2, 0, 1)), np.transpose(d[n], (2, 0, 1)))
            w, b = w + gw, b + gb
        out += [np.transpose(w, (2, 3, 0, 1)).reshape(9, 32, -1), b]
    return out


def _close(got, want, magnitude):
    assert (np.abs(got.astype(np.float64) - want) <= DEPTH * 2.0**-24 * magnitude + 1e-38).all()


@pytest.mark.parametrize("channels", [32, 4])
@pytest.mark.parametrize("shape", SHAPES)
def test_both_gradients(shape, channels):
    N, H, W = shape
    rng = np.random.Generator(np.random.PCG64(H * W + channels))
    xb, x64 = bf16(np.maximum(rng.standard_normal((N, H, W, 32)), 0.0))
    real = 3 if channels == 4 else 32
    dy = np.zeros((N, H, W, 32))
    dy[..., :real] = 0.1 * rng.standard_normal((N, H, W, real))
    dyb, dy64 = bf16(dy)
    given = dyb[..., :channels].contiguous()
    wd, _ = bf16(0.1 * rng.standard_normal((9, 32, 32)))
    want_dx = torch.empty_like(xb)
    check(lib().sw2d_conv3x3_dgrad(ptr(dyb), ptr(wd), ptr(xb), ptr(want_dx), N, H, W, stream()))
    want_w, want_b, mag_w, mag_b = _oracle(x64, dy64)
    # the room that the size function states, and the least that is accepted (fewer workgroups)
    full = lib().sw2d_wgrad_workspace_bytes(32, N, H, W)
    least = (-(-W // 128) * -(-H // 4) * N + 7) // 8 * (9 * 32 * 32 + 32) * 4
    for need in (full, least):
        work = torch.full((need,), 0xFF, dtype=torch.uint8, device=DEV)
        dx = torch.full_like(xb, float("nan"))
        dW = torch.full((9, 32, 32), float("nan"), dtype=torch.float32, device=DEV)
        db = torch.full((32,), float("nan"), dtype=torch.float32, device=DEV)
        check(lib().sw2d_conv3x3_backward(ptr(xb), ptr(given), channels, ptr(wd), ptr(dx), N, H, W, ptr(dW), ptr(db),
                                          ptr(work), need, stream()))
        assert torch.equal(dx, want_dx)
        _close(dW.cpu().numpy(), want_w, mag_w)
        _close(db.cpu().numpy(), want_b, mag_b)
    assert lib().sw2d_conv3x3_backward(ptr(xb), ptr(given), channels, ptr(wd), ptr(dx), N, H, W, ptr(dW), ptr(db),
                                       ptr(work), least - 1, stream()) == _lib.SW2D_ENOSPC


@pytest.mark.parametrize("cin", [16, 32])
@pytest.mark.parametrize("shape", SHAPES)
def test_weight_gradient_alone(shape, cin):
    N, H, W = shape
    rng = np.random.Generator(np.random.PCG64(H * W + cin))
    xb, x64 = bf16(rng.standard_normal((N, H, W, cin)))
    dyb, dy64 = bf16(0.1 * rng.standard_normal((N, H, W, 32)))
    need = lib().sw2d_wgrad_workspace_bytes(cin, N, H, W)
    work = torch.full((need,), 0xFF, dtype=torch.uint8, device=DEV)
    dW = torch.empty((9, 32, cin), dtype=torch.float32, device=DEV)
    db = torch.empty(32, dtype=torch.float32, device=DEV)
    check(lib().sw2d_conv3x3_wgrad(ptr(xb), cin, ptr(dyb), N, H, W, ptr(dW), ptr(db), ptr(work), need, stream()))
    want_w, want_b, mag_w, mag_b = _oracle(x64, dy64)
    _close(dW.cpu().numpy(), want_w, mag_w)
    _close(db.cpu().numpy(), want_b, mag_b)


@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 7, 9), (2, 23, 31), (1, 64, 64)])
def test_four_channel_loss_gradient_equals_the_padded_one(shape):
    N, H, W = shape
    rng = np.random.Generator(np.random.PCG64(H * W))
    out, tgt = (torch.from_numpy(rng.standard_normal((N, 3, H, W)).astype(np.float32)).to(DEV) for _ in range(2))
    mask = torch.from_numpy((rng.uniform(size=(N, H, W)) < 0.8).astype(np.uint8)).to(DEV)
    scale = np.array([2.0, 0.5, 1.0], dtype=np.float32)
    sp = scale.ctypes.data_as(ctypes.POINTER(ctypes.c_float))
    wb = lib().sw2d_mse_workspace_bytes()
    work = torch.empty(wb, dtype=torch.uint8, device=DEV)
    got = []
    for name, channels in (("sw2d_mse_grad", 32), ("sw2d_mse_grad4", 4)):
        d = torch.full((N, H, W, channels), float("nan"), dtype=torch.bfloat16, device=DEV)
        loss = torch.zeros(1, dtype=torch.float64, device=DEV)
        check(getattr(lib(), name)(ptr(out), ptr(tgt), sp, ptr(mask), N, H, W, ctypes.c_float(0.125), ptr(d), ptr(loss),
                                   ptr(work), wb, stream()))
        got.append((d, loss.item()))
    assert torch.equal(got[0][0][..., :4], got[1][0]) and not got[0][0][..., 3:].any()
    assert got[0][1] == got[1][1]


def test_network_adam_equals_adam_then_casts():
    from paper_1711_04471_amd import surrogate as S
    a, b = S.ConvNet(seed=3), S.ConvNet(seed=3)
    gen = torch.Generator(device=DEV).manual_seed(1)
    for t in range(1, 4):
        a.grad.copy_(torch.randn(a.n_params, generator=gen, device=DEV))
        b.grad.copy_(a.grad)
        a.adam(lr=1e-2)
        check(lib().sw2d_adam(ptr(b.theta), ptr(b.grad), ptr(b.m), ptr(b.v), b.n_params, t, ctypes.c_float(1e-2),
                              ctypes.c_float(0.9), ctypes.c_float(0.999), ctypes.c_float(1e-8), stream()))
        b.cast()
    for x, y in zip([a.theta, a.m, a.v, *a.wk, *a.wd[1:]], [b.theta, b.m, b.v, *b.wk, *b.wd[1:]]):
        assert torch.equal(x, y)


@pytest.mark.parametrize("channels", [32, 4])
def test_very_wide_image(channels):
    """Rows longer than a tile's 32-bit byte offsets reach; pixels that count lie at both ends."""
    N, H, W, edge = 1, 2, 932100, 40
    rng = np.random.Generator(np.random.PCG64(channels))
    x = torch.zeros((N, H, W, 32), dtype=torch.bfloat16, device=DEV)
    dy = torch.zeros_like(x)
    wants = None
    for side in (slice(0, edge), slice(W - edge, W)):
        xb, x64 = bf16(np.maximum(rng.standard_normal((N, H, edge, 32)), 0.0))
        d = np.zeros((N, H, edge, 32))
        d[..., :3] = 0.1 * rng.standard_normal((N, H, edge, 3))
        db_, d64 = bf16(d)
        x[:, :, side], dy[:, :, side] = xb, db_
        got = _oracle(x64, d64)
        wants = got if wants is None else [p + q for p, q in zip(wants, got)]
    given = dy[..., :channels].contiguous()
    wd, _ = bf16(0.1 * rng.standard_normal((9, 32, 32)))
    want_dx, dx = torch.empty_like(x), torch.full_like(x, float("nan"))
    check(lib().sw2d_conv3x3_dgrad(ptr(dy), ptr(wd), ptr(x), ptr(want_dx), N, H, W, stream()))
    need = lib().sw2d_wgrad_workspace_bytes(32, N, H, W)
    work = torch.empty(need, dtype=torch.uint8, device=DEV)
    dW = torch.empty((9, 32, 32), dtype=torch.float32, device=DEV)
    db = torch.empty(32, dtype=torch.float32, device=DEV)
    check(lib().sw2d_conv3x3_backward(ptr(x), ptr(given), channels, ptr(wd), ptr(dx), N, H, W, ptr(dW), ptr(db),
                                      ptr(work), need, stream()))
    assert torch.equal(dx, want_dx)
    _close(dW.cpu().numpy(), wants[0], wants[2])
    _close(db.cpu().numpy(), wants[1], wants[3])
    check(lib().sw2d_conv3x3_wgrad(ptr(x), 32, ptr(dy), N, H, W, ptr(dW), ptr(db), ptr(work), need, stream()))
    _close(dW.cpu().numpy(), wants[0], wants[2])
