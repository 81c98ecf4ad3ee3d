"""Register tiles against the streamed row pipelines: the same state bit for bit, the same
maxima, the volumes up to the order of their sums, at the edges of the tiles' sizes."""
import ctypes

import numpy as np
import pytest

from paper_1711_04471_amd import inputs

pytestmark = pytest.mark.gpu

# a tile is 128 columns x 24 or 40 rows; neighbours overlap by 4 K columns and rows
EDGES = [(3, 3), (66, 66), (127, 23), (128, 24), (129, 25), (240, 32), (241, 33), (113, 40), (116, 44), (352, 41)]


def _run(case, calls, streaming, spp=1, rows=8):
    from paper_1711_04471_amd.sw2d import Sw2d
    with Sw2d.from_case(case) as sim:
        sim.streaming = streaming
        assert sim.streaming == streaming
        if spp > 1:
            sim.set_time_blocking(spp, rows=min(rows, case.ny))
        for n in calls:
            sim.step(n)
        return sim.state_numpy(), sim.reduce(sum(calls))


def _same(a, b, case):
    for x, y in zip(a[0], b[0]):
        assert np.array_equal(x, y, equal_nan=True)
    assert np.array_equal(a[1]["step"], b[1]["step"])
    for name in ("max_abs_u", "max_abs_v"):
        assert np.array_equal(a[1][name], b[1][name])
    # sums of the same FP32 surfaces in FP64, in another order
    atol = 1e-12 * case.dx * case.dy * max(1.0, float(np.abs(case.eta).sum(dtype=np.float64)))
    for name in ("vol_total", "vol_disp"):
        np.testing.assert_allclose(a[1][name], b[1][name], rtol=1e-12, atol=atol)


@pytest.mark.parametrize("shape", EDGES)
def test_tiles_equal_streamed_steps(shape):
    nx, ny = shape
    if shape == (3, 3):
        c = inputs.gaussian_basin_64()
        sl = slice(31, 34)
        for name in ("H", "eta", "u", "v", "mask"):
            setattr(c, name, getattr(c, name)[sl, sl].copy())
        c.nx = c.ny = 3
        c.mask[:] = 0
        c.mask[1, 1] = 1
        c.eta[c.mask == 0] = 0.0
    else:
        c = inputs.small_basin(nx, ny, seed=nx + ny)
    want = _run(c, [21], True)
    for calls in ([21], [1, 2, 3, 4, 11], [1] * 5 + [16]):
        _same(_run(c, calls, False), want, c)


@pytest.mark.parametrize("shape", [(693, 700), (701, 523), (1024, 1000)])
def test_tall_tiles_equal_streamed_steps(shape):
    """Grids with more than 320 low tiles at 2, 3 and 4 steps per pass (40-row tiles)."""
    c = inputs.small_basin(*shape, seed=sum(shape))
    want = _run(c, [13], True)
    for calls in ([13], [2, 3, 8]):
        _same(_run(c, calls, False), want, c)


@pytest.mark.parametrize("spp", [2, 3, 4])
@pytest.mark.parametrize("shape,nsteps", [((700, 530), 37), ((61, 47), 20), ((300, 1201), 9), ((113, 40), 13),
                                          ((234, 41), 11)])
def test_streamed_k_steps_equal_tiles(shape, nsteps, spp):
    c = inputs.small_basin(*shape, seed=sum(shape))
    want = _run(c, [nsteps], False)
    for rows in (8, 32, 64):
        _same(_run(c, [nsteps], True, spp, rows), want, c)


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
def test_non_finite_states_spread_alike(bad):
    """A non-finite surface or velocity set between steps reaches the same cells, and the folds
    report it."""
    from paper_1711_04471_amd import _lib
    from paper_1711_04471_amd.sw2d import Sw2d
    c = inputs.small_basin(150, 61, seed=5)
    j, i = [int(x) for x in np.argwhere(c.mask[8:-8, 8:-8] != 0)[1234] + 8]
    got = []
    for streaming in (True, False):
        with Sw2d.from_case(c) as sim:
            sim.streaming = streaming
            e, u, v = (a.copy() for a in (c.eta, c.u, c.v))
            e[j, i] = bad
            sim.set_state(e, u, v)
            sim.step(3)
            with pytest.raises(_lib.Sw2dError) as err:
                sim.reduce(1)
            assert err.value.code == _lib.SW2D_EUNSTABLE
            got.append(sim.state_numpy())
    for x, y in zip(*got):
        assert np.array_equal(x, y, equal_nan=True)


def test_state_off_8_bytes_steps_alike():
    """The caller's state need only be aligned to its floats: one that is not on 8 bytes takes the
    4-byte accesses."""
    import torch

    from paper_1711_04471_amd import _lib
    from paper_1711_04471_amd.sw2d import params
    c = inputs.small_basin(130, 70, seed=9)
    want = _run(c, [6], True)
    L = _lib.load()
    n = c.nx * c.ny
    buf = torch.zeros(6 * n + 1, device="cuda")
    for f, a in enumerate((c.eta, c.u, c.v)):
        buf[1 + f * n:1 + (f + 1) * n] = torch.from_numpy(a.reshape(-1)).cuda()
    H, mask = torch.from_numpy(c.H).cuda(), torch.from_numpy(c.mask).cuda()
    p = params(c.nx, c.ny, c.dx, c.dy, c.g, c.dt, c.eps)
    nb = L.sw2d_workspace_bytes(ctypes.byref(p))
    work = torch.empty(nb, dtype=torch.uint8, device="cuda")
    h = ctypes.c_void_p()
    s = torch.cuda.current_stream()
    assert L.sw2d_create(ctypes.byref(p), H.data_ptr(), mask.data_ptr(), buf.data_ptr() + 4, work.data_ptr(), nb,
                         s.cuda_stream, ctypes.byref(h)) == 0
    assert L.sw2d_step(h, 6) == 0
    ptr = ctypes.c_void_p()
    assert L.sw2d_state(h, ctypes.byref(ptr), None, None) == 0
    torch.cuda.synchronize()
    off = (ptr.value - buf.data_ptr()) // 4
    assert np.array_equal(buf[off:off + n].cpu().numpy().reshape(c.ny, c.nx), want[0][0])
    L.sw2d_destroy(h)


def _variant_state(case, flags, calls, streaming, spp=1):
    from paper_1711_04471_amd.sw2d import Sw2d
    with Sw2d.from_case(case, flags=flags, cd=0.0025, hmin=0.0625) as sim:
        sim.streaming = streaming
        if spp > 1:
            sim.set_time_blocking(spp, rows=min(8, case.ny))
        for n in calls:
            sim.step(n)
        return sim.state_numpy(), sim.reduce(sum(calls))


def _variant_case(shape, flags):
    make = inputs.shore_basin if flags == 8 else inputs.small_basin
    return make(*shape, seed=sum(shape) + flags)


# 24-row tiles; 40-row tiles; 64-row tiles at 4 steps per pass; two steps per pass with friction
@pytest.mark.parametrize("shape", [(66, 66), (117, 33), (251, 61), (693, 700), (1024, 1000), (2047, 1100)])
@pytest.mark.parametrize("flags", [1, 2, 3, 4, 5, 6, 7, 8])
def test_variant_tiles_equal_streamed_steps(flags, shape):
    c = _variant_case(shape, flags)
    calls = [1, 2, 3, 15]
    _same(_variant_state(c, flags, calls, False), _variant_state(c, flags, calls, True), c)


@pytest.mark.parametrize("flags", [0, 2, 7, 8])
def test_grids_past_the_cache_equal_streamed_steps(flags):
    """More than 2^23 cells: 64-row tiles, the caller's steps per pass where one is chosen."""
    c = _variant_case((3001, 2900), flags)
    _same(_variant_state(c, flags, [1, 2, 3, 4], False), _variant_state(c, flags, [1, 2, 3, 4], True), c)
    if not flags & 4:
        _same(_variant_state(c, flags, [7], False, 3), _variant_state(c, flags, [7], True), c)
