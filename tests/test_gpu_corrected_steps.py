"""Corrected steps whose correction is added as the step stores its state, against the network, the step
and the correction as three calls: bitwise the same state and diagnostics, at the edges of the tiles."""
import ctypes

import numpy as np
import pytest
import torch

from paper_1711_04471_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(5, 7), (66, 66), (127, 21), (128, 20), (129, 41), (124, 24), (253, 43), (301, 221)])
def test_advance_equals_three_calls(shape):
    from paper_1711_04471_amd import surrogate as S
    from paper_1711_04471_amd._lib import check
    from paper_1711_04471_amd.sw2d import Sw2d
    nx, ny = shape
    c = inputs.small_basin(nx, ny, seed=nx + ny)
    net = S.ConvNet(seed=5)
    H = torch.as_tensor(c.H).cuda()
    mask = torch.as_tensor(c.mask).cuda()
    _, mp = S._fptr(np.array([0.02, 0.0, 0.0, 27.0, 0.9], np.float32))
    _, sp = S._fptr(np.array([0.2, 0.1, 0.1, 10.0, 0.3], np.float32))
    keep, tp = S._fptr(np.array([2e-3, 1e-3, 3e-3], np.float32))
    calls, steps = [2, 1, 3], 6

    def p(t):
        return ctypes.c_void_p(t.data_ptr())

    with Sw2d.from_case(c) as a, Sw2d.from_case(c) as b, Sw2d.from_case(c) as w:
        w.streaming = True
        for _ in range(steps):
            out = net.forward_fused(*a.state(), H, mask, ny, nx, mp, sp)
            a.step(1)
            e, u, v = a.state()
            check(net.lib.sw2d_apply_correction(p(e), p(u), p(v), p(out), p(mask), nx, ny, tp, net.stream()), "correct")
        want, folds = a.state_numpy(), a.reduce(steps)
        plain = Sw2d.from_case(c)
        plain.step(steps)
        assert not np.array_equal(plain.state_numpy()[0], want[0])  # the correction is seen
        plain.close()
        for n in calls:
            net.advance(b, n, H, mask, mp, sp, tp)
            net.advance(w, n, H, mask, mp, sp, tp)
        for x, y, z in zip(want, b.state_numpy(), w.state_numpy()):
            assert np.array_equal(x, y) and np.array_equal(x, z)
        got = b.reduce(steps)
        for name in ("step", "vol_total", "vol_disp", "max_abs_u", "max_abs_v"):
            assert np.array_equal(folds[name], got[name])  # same tiles, same order of the sums
