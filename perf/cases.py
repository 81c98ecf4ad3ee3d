"""Performance cases: the work that a program using this package has it do, at the sizes of the
repository's own workloads and over the ranges around them.

``listed()`` names the fixed cases, ``draw(rng)`` gives one more of the same ranges,
``prepare(case, seed)`` makes what a program holds before the call (inputs from the seed, the
handle it keeps), ``run(state)`` is one pass through the public entry points, ``work(case)`` its
unavoidable bytes and operations and ``exact(case, seed)`` its outputs in 64 bits from plain torch.

Kinds of cases:

* ``step``: a closed basin advanced by ``Sw2d.step`` (one step per pass or several, plain or with
  model variants). Real use: the time loop between two outputs of the model.
* ``ensemble``: uneven basins advanced together by ``Sw2dBatch.step``, their states gathered into
  one array per field. Real use: an ensemble run between two outputs.
* ``corrected``: the learned coarse model: network, coarse steps, correction, as the rollout
  sequences them (the correction before every m-th step, or before every step by
  ``ConvNet.advance``). Real use: inference.
* ``train``: one minibatch of the network's training: forward, masked loss, backward, Adam.
* ``judge``: the fine state restricted to the coarse grid and the RMSE of the coarse surface
  against it. Real use: each check of the learned model against the fine one.
* ``sor``: a pressure solve by red-black SOR with its residual history. Real use: one time step's
  pressure solve of the paper's second workload.
"""

from __future__ import annotations

import ctypes
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_1711_04471_amd import _lib, surrogate
from paper_1711_04471_amd._lib import check
from paper_1711_04471_amd.sw2d import ADVECTION, FILTER_UV, FRICTION, WETDRY, SorSolver, Sw2d, Sw2dBatch

G = 9.81
EPS = 0.05
DX = 500.0
CD = 0.0025
HMIN = 0.0625
DEEPEST = 50.0  # m: depths lie in 5..50 m
DT = 0.5 * DX / math.sqrt(G * DEEPEST)

# typical normalisation of the network's inputs (eta, u, v, H, mask) and scale of its correction
IN_MEAN = (0.02, 0.0, 0.0, 27.0, 0.9)
IN_STD = (0.2, 0.1, 0.1, 10.0, 0.3)
T_STD = (2e-5, 1e-5, 1e-5)
LR = 1e-3
NOISE = 0.3  # Trainer's default input noise


def listed():
    return [
        # the 64 x 64 basin with its land border, 200 steps: the smallest time loop
        {"name": "step_66", "kind": "step", "nx": 66, "ny": 66, "steps": 200, "per_pass": 1, "rows": 0, "flags": 0},
        # an ordinary basin, one step per pass, as a handle steps by default
        {"name": "step_2048", "kind": "step", "nx": 2048, "ny": 2048, "steps": 50, "per_pass": 1, "rows": 0,
         "flags": 0},
        # the largest basin, four steps per pass on 128-row bands, as the benchmark steps it
        {"name": "step_8192_k4", "kind": "step", "nx": 8192, "ny": 8192, "steps": 20, "per_pass": 4, "rows": 128,
         "flags": 0},
        # an odd width with friction, velocity filter and momentum advection together
        {"name": "step_all_variants", "kind": "step", "nx": 2047, "ny": 1531, "steps": 20, "per_pass": 1, "rows": 0,
         "flags": FRICTION | FILTER_UV | ADVECTION},
        # the benchmark's ensemble: 256 uneven members, three steps per pass
        {"name": "ensemble_256", "kind": "ensemble", "members": 256, "lo": 128, "hi": 1024, "steps": 48,
         "per_pass": 3, "rows": 64},
        # a dozen small members with the library's defaults: latency counts
        {"name": "ensemble_12", "kind": "ensemble", "members": 12, "lo": 64, "hi": 256, "steps": 50, "per_pass": 1,
         "rows": 0},
        # the judged rollout's inner loop on the 1024 x 1024 coarse grid: network before every 5th step
        {"name": "corrected_1024", "kind": "corrected", "nx": 1024, "ny": 1024, "rounds": 4, "every": 5},
        # a small, odd coarse grid corrected at every step
        {"name": "corrected_300x221", "kind": "corrected", "nx": 300, "ny": 221, "rounds": 5, "every": 1},
        # the training minibatch of the coarse grid
        {"name": "train_4x1024", "kind": "train", "nx": 1024, "ny": 1024, "batch": 4},
        # a check of the 1024 x 1024 coarse model against its 4096 x 4096 fine model
        {"name": "judge_4096", "kind": "judge", "nx": 4096, "ny": 4096},
        # the large-eddy simulator's pressure grid, 50 iterations
        {"name": "sor_300x300x90", "kind": "sor", "nx": 300, "ny": 300, "nz": 90, "iters": 50, "fused": 0},
        # a small pressure grid of odd sides
        {"name": "sor_65x47x33", "kind": "sor", "nx": 65, "ny": 47, "nz": 33, "iters": 50, "fused": 0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "ensemble", "corrected", "train", "judge", "sor"])
    if kind == "step":
        nx, ny = _log_int(rng, 40, 6000), _log_int(rng, 40, 6000)
        per_pass = rng.choice([1, 1, 2, 3, 4])
        flags = rng.choice([0, 0, 0, FRICTION, FILTER_UV, FRICTION | FILTER_UV, WETDRY])
        if per_pass == 1:
            flags = rng.choice([flags, flags, ADVECTION, FRICTION | FILTER_UV | ADVECTION])
        rows = 0 if per_pass == 1 else min(ny, rng.choice([8, 16, 32, 48, 64, 128]))
        return {"kind": kind, "nx": nx, "ny": ny, "steps": rng.randint(4, 48), "per_pass": per_pass, "rows": rows,
                "flags": flags}
    if kind == "ensemble":
        members = _log_int(rng, 4, 96)
        lo = rng.choice([40, 64, 128])
        per_pass = rng.choice([1, 2, 3])
        return {"kind": kind, "members": members, "lo": lo, "hi": rng.choice([256, 512, 1024]),
                "steps": 6 * rng.randint(2, 6), "per_pass": per_pass, "rows": rng.choice([0, 16, 32])}
    if kind == "corrected":
        return {"kind": kind, "nx": _log_int(rng, 60, 1400), "ny": _log_int(rng, 60, 1400),
                "rounds": rng.randint(2, 6), "every": rng.choice([1, 5, 10])}
    if kind == "train":
        return {"kind": kind, "nx": _log_int(rng, 64, 1024), "ny": _log_int(rng, 64, 1024),
                "batch": rng.choice([1, 2, 4])}
    if kind == "judge":
        return {"kind": kind, "nx": 4 * _log_int(rng, 30, 1200), "ny": 4 * _log_int(rng, 30, 1200)}
    return {"kind": "sor", "nx": _log_int(rng, 20, 320), "ny": _log_int(rng, 20, 320), "nz": _log_int(rng, 10, 120),
            "iters": rng.choice([20, 50]), "fused": rng.choice([0, 0, 1])}


# ------------------------------------------------------------------------------------ inputs
def _generator(seed, *tags):
    return np.random.Generator(np.random.PCG64([int(seed), *(int(t) for t in tags)]))


def _cuda64(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64).cuda()


def _modes(rng, nx, ny, n=16):
    """A smooth field of n random Fourier modes (|k| <= 4), scaled to [0, 1]."""
    kx, ky = rng.integers(-4, 5, n), rng.integers(1, 5, n)
    amp = rng.standard_normal(n) / np.hypot(kx, ky)
    ax = 2.0 * np.pi * np.outer(kx, (np.arange(nx) + 0.5) / nx) + rng.uniform(0.0, 2.0 * np.pi, n)[:, None]
    by = 2.0 * np.pi * np.outer(ky, (np.arange(ny) + 0.5) / ny)
    left = np.concatenate([np.cos(by).T * amp, -np.sin(by).T * amp], axis=1)
    right = np.concatenate([np.cos(ax), np.sin(ax)], axis=0)
    b = _cuda64(left) @ _cuda64(right)
    return (b - b.min()) / (b.max() - b.min())


def _mask(rng, nx, ny, border):
    """A land border and disks of land over about a tenth of the interior (uint8, host)."""
    mask = np.zeros((ny, nx), dtype=np.uint8)
    mask[border:ny - border, border:nx - border] = 1
    side = min(nx, ny)
    for _ in range(int(48 * max(nx, ny) / side)):
        cx, cy, r = rng.uniform(0, nx), rng.uniform(0, ny), rng.uniform(0.01, 0.04) * side
        i0, i1 = max(0, int(cx - r) - 1), min(nx, int(cx + r) + 2)
        j0, j1 = max(0, int(cy - r) - 1), min(ny, int(cy + r) + 2)
        inside = (np.arange(i0, i1) + 0.5 - cx)[None, :] ** 2 + (np.arange(j0, j1) + 0.5 - cy)[:, None] ** 2 <= r * r
        mask[j0:j1, i0:i1][inside] = 0
    return mask


def _bumps(rng, nx, ny, n):
    """n Gaussian surface bumps of 0.1..1 m, sigma 8..32 cells."""
    a, s = rng.uniform(0.1, 1.0, n), rng.uniform(8.0, 32.0, n)
    cx, cy = rng.uniform(0.0, nx, n), rng.uniform(0.0, ny, n)
    gx = np.exp(-((np.arange(nx) + 0.5)[None, :] - cx[:, None]) ** 2 / (2.0 * s[:, None] ** 2))
    gy = np.exp(-((np.arange(ny) + 0.5)[None, :] - cy[:, None]) ** 2 / (2.0 * s[:, None] ** 2))
    return _cuda64((gy * a[:, None]).T) @ _cuda64(gx)


def _basin(nx, ny, seed, n_bumps=8, border=1, shore=False, scale=1.0):
    """A seeded closed basin on the GPU: smooth depth, land disks, a bumpy surface at rest. With
    ``shore`` the depth ramps up to dry ground in the east and the still water stands 1 m low."""
    rng = _generator(seed, nx, ny)
    H = 5.0 + (DEEPEST - 5.0) * _modes(rng, nx, ny)
    mask = torch.from_numpy(_mask(rng, nx, ny, border)).cuda()
    eta = _bumps(rng, nx, ny, n_bumps)
    if shore:
        x = (torch.arange(nx, dtype=torch.float64, device="cuda") + 0.5) / nx
        H = 0.2 + (H - 0.2) * ((0.95 - x) / 0.35).clamp(0.0, 1.0)[None, :]
        eta = torch.where(H > 1.0, eta - 1.0, -H)
    H = H.float()
    eta = torch.where(mask != 0, eta.float(), 0.0)
    if shore:
        eta = torch.maximum(eta, torch.where(mask != 0, -H, 0.0))
    z = torch.zeros_like(H)
    return SimpleNamespace(nx=nx, ny=ny, dx=DX * scale, dy=DX * scale, g=G, dt=DT * scale, eps=EPS, H=H, mask=mask,
                           eta=eta, u=z, v=z)


def _members(case, seed):
    rng = _generator(seed, case["members"], case["lo"], case["hi"])
    # the sides are the case's own (the same work for every seed), the basins the seed's
    sides = _generator(0, case["members"], case["lo"], case["hi"]).integers(case["lo"], case["hi"] + 1,
                                                                          (case["members"], 2))
    return [_basin(int(a), int(b), int(rng.integers(1 << 30)), n_bumps=int(rng.integers(1, 5))) for a, b in sides]


def _floats(values):
    return (ctypes.c_float * len(values))(*values)


def _net(seed):
    """A network whose last layer gives outputs of order one, as a trained one's."""
    net = surrogate.ConvNet(seed=seed)
    w, _ = net.weight(3)
    w *= 3.0
    for layer in range(4):
        b = net.weight(layer)[1]
        real = surrogate.REAL_OUT[layer]
        b[:real] = torch.from_numpy(_generator(seed, 7, layer).uniform(-0.1, 0.1, real)).float().cuda()
    net.cast()
    return net


def _dataset(case, seed):
    """Eight snapshot pairs of two basins, with fields of the scales that the normalisation states."""
    nx, ny, samples = case["nx"], case["ny"], 8
    basins = [_basin(nx, ny, seed * 2 + r, border=1) for r in range(2)]
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    rnd = lambda *shape: torch.randn(shape, generator=gen, device="cuda")  # noqa: E731
    run_of = np.repeat(np.arange(2), samples // 2)
    wet = torch.stack([b.mask for b in basins]).float()[torch.as_tensor(run_of).cuda()]
    scale = torch.tensor(IN_STD[:3], device="cuda")[:, None, None, None]
    inputs = rnd(3, samples, ny, nx) * scale * wet
    targets = rnd(3, samples, ny, nx) * torch.tensor(T_STD, device="cuda")[:, None, None, None] * wet
    stats = surrogate.Stats(np.array(IN_MEAN, np.float32), np.array(IN_STD, np.float32), np.array(T_STD, np.float32))
    return surrogate.Dataset(inputs, targets, run_of, torch.stack([b.H for b in basins]),
                             torch.stack([b.mask for b in basins]), stats)


def _moments(net, seed):
    """Adam's moments of a network in the middle of its training (zero on the padding weights)."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed) + 1)
    real = (net.theta != 0).float()
    return (torch.randn(net.n_params, generator=gen, device="cuda") * 3e-3 * real,
            (1e-2 * (0.5 + torch.rand(net.n_params, generator=gen, device="cuda"))) ** 2 * real)


def _poisson(case, seed):
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    rng = _generator(seed, nx, ny, nz)
    axes = [np.arange(n, dtype=np.float64) for n in (nz, ny, nx)]
    f = torch.zeros((nz, ny, nx), dtype=torch.float64, device="cuda")
    for _ in range(8):
        widths = (rng.uniform(3.0, 12.0), rng.uniform(5.0, 20.0), rng.uniform(5.0, 20.0))
        gz, gy, gx = (_cuda64(np.exp(-0.5 * ((a - rng.uniform(0, len(a))) / s) ** 2)) for a, s in zip(axes, widths))
        f += rng.uniform(-1.0, 1.0) * gz[:, None, None] * gy[None, :, None] * gx[None, None, :]
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    f = (f + 1e-3 * (2.0 * torch.rand(f.shape, generator=gen, device="cuda", dtype=torch.float64) - 1.0)).float()
    p = 0.1 * torch.randn(f.shape, generator=gen, device="cuda")  # the last time step's pressure
    return p, f


# ------------------------------------------------------------------------------------ prepare
def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind == "step":
        flags = case["flags"]
        b = _basin(case["nx"], case["ny"], seed, shore=bool(flags & WETDRY))
        s["sim"] = Sw2d.from_case(b, flags=flags, cd=CD if flags & FRICTION else 0.0,
                                  hmin=HMIN if flags & WETDRY else 0.0)
        if case["per_pass"] > 1:
            s["sim"].set_time_blocking(case["per_pass"], rows=case["rows"])
    elif kind == "ensemble":
        members = _members(case, seed)
        rows = [min(case["rows"], m.ny) for m in members] if case["rows"] else None
        s["batch"] = Sw2dBatch(members, band_rows=rows)
        s["batch"].set_time_blocking(case["per_pass"])
    elif kind == "corrected":
        b = _basin(case["nx"], case["ny"], seed, scale=4.0)
        s["basin"], s["net"] = b, _net(seed)
        s["sim"] = Sw2d.from_case(b)
        s["sim"].set_time_blocking(3, rows=8)
        s["mean"], s["std"], s["t_std"] = _floats(IN_MEAN), _floats(IN_STD), _floats(T_STD)
    elif kind == "train":
        ds = _dataset(case, seed)
        net = _net(seed)
        m, v = _moments(net, seed)
        net.m.copy_(m)
        net.v.copy_(v)
        net.t = 100
        s["trainer"] = surrogate.Trainer(net, ds, batch=case["batch"], noise=NOISE)
        s["next"] = 0
    elif kind == "judge":
        b = _basin(case["nx"], case["ny"], seed, border=4)
        s["fine"] = Sw2d.from_case(b)
        s["coarse"] = co = surrogate.Coarse(s["fine"], b)
        s["fine"].step(8)
        co.sim.step(2)
        s["ref"] = [torch.empty_like(t) for t in (co.eta, co.u, co.v, co.H, co.mask)]
    else:
        s["p"], s["f"] = _poisson(case, seed)
        s["solver"] = SorSolver(case["nx"], case["ny"], case["nz"], 4.0, 4.0, 2.0, 1.7, case["iters"],
                                fused=bool(case["fused"]))
    return s


# ------------------------------------------------------------------------------------ run
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "step":
        s["sim"].step(case["steps"])
        return dict(zip(("eta", "u", "v"), s["sim"].state()))
    if kind == "ensemble":
        s["batch"].step(case["steps"])
        states = [s["batch"].state(k) for k in range(case["members"])]
        return {name: torch.cat([st[f].reshape(-1) for st in states]) for f, name in enumerate(("eta", "u", "v"))}
    if kind == "corrected":
        sim, net, b = s["sim"], s["net"], s["basin"]
        if case["every"] == 1:
            net.advance(sim, case["rounds"], b.H, b.mask, s["mean"], s["std"], s["t_std"])
            return dict(zip(("eta", "u", "v"), sim.state()))
        lib, stream = _lib.load(), torch.cuda.current_stream().cuda_stream
        for _ in range(case["rounds"]):
            e, u, v = sim.state()
            out = net.forward_fused(e, u, v, b.H, b.mask, sim.ny, sim.nx, s["mean"], s["std"])
            sim.step(case["every"])
            e, u, v = sim.state()
            check(lib.sw2d_apply_correction(e.data_ptr(), u.data_ptr(), v.data_ptr(), out.data_ptr(),
                                            b.mask.data_ptr(), sim.nx, sim.ny, s["t_std"], stream),
                  "sw2d_apply_correction")
        return {"eta": e, "u": u, "v": v, "out": out}
    if kind == "train":
        t, n = s["trainer"], case["batch"]
        first = s["next"] * n % 8
        s["next"] += 1
        t.step(range(first, first + n))
        t.net.adam(lr=LR)
        return {"loss": t.loss, "grad": t.net.grad, "theta": t.net.theta, "m": t.net.m, "v": t.net.v}
    if kind == "judge":
        co = s["coarse"]
        co.restrict(s["fine"], out=s["ref"])
        rmse = co.rmse_eta(s["ref"][0])
        return {"eta": s["ref"][0], "u": s["ref"][1], "v": s["ref"][2], "H": s["ref"][3], "mask": s["ref"][4],
                "rmse": rmse}
    s["solver"].run(s["p"], s["f"])
    res = s["solver"].res
    return {"p": s["p"], "max_abs_r": res.view(torch.float32)[1::4], "sum_r2": res.view(torch.float64)[1::2]}


# ------------------------------------------------------------------------------------ work
def work(case):
    kind = case["kind"]
    if kind == "step":
        cells = case["nx"] * case["ny"]
        flags = case["flags"]
        ops = 33 + (8 if flags & FRICTION else 0) + (22 if flags & FILTER_UV else 0) + (30 if flags & ADVECTION else 0)
        return {"bytes": 28.0 * cells, "flops": float(ops) * cells * case["steps"]}
    if kind == "ensemble":
        sides = _generator(0, case["members"], case["lo"], case["hi"]).integers(case["lo"], case["hi"] + 1,
                                                                              (case["members"], 2))
        cells = float((sides[:, 0] * sides[:, 1]).sum())
        # the step, then the states gathered
        return {"bytes": (28.0 + 24.0) * cells, "flops": 33.0 * cells * case["steps"]}
    if kind == "corrected":
        cells = case["nx"] * case["ny"]
        return {"bytes": 41.0 * cells, "flops": case["rounds"] * (41472.0 + 33.0 * case["every"]) * cells}
    if kind == "train":
        cells = case["nx"] * case["ny"] * case["batch"]
        return {"bytes": 29.0 * cells, "flops": 121536.0 * cells}
    if kind == "judge":
        cells = case["nx"] * case["ny"]
        return {"bytes": (17.0 + 26.0 / 16.0) * cells, "flops": 4.0 * cells}
    cells = case["nx"] * case["ny"] * case["nz"]
    return {"bytes": 12.0 * cells, "flops": 16.0 * cells * case["iters"]}


# ------------------------------------------------------------------------------------ exact
def _shift(a, dj, di):
    """a[j + dj, i + di], zero (false) off the grid."""
    out = torch.zeros_like(a)
    ny, nx = a.shape
    src = a[max(dj, 0):ny + min(dj, 0), max(di, 0):nx + min(di, 0)]
    out[max(-dj, 0):ny + min(-dj, 0), max(-di, 0):nx + min(-di, 0)] = src
    return out


def _filtered(x, active, eps):
    s = torch.zeros_like(x)
    for dj, di in ((0, 1), (0, -1), (1, 0), (-1, 0)):
        s += torch.where(_shift(active, dj, di), _shift(x, dj, di) - x, 0.0)
    return torch.where(active, x + eps / 4.0 * s, 0.0)


def _exact_step(e, u, v, h, w, wx, wy, b, flags):
    """One time step in 64 bits; w, wx, wy: water cells, active east faces, active north faces."""
    east, west = (lambda a: _shift(a, 0, 1)), (lambda a: _shift(a, 0, -1))
    north, south = (lambda a: _shift(a, 1, 0)), (lambda a: _shift(a, -1, 0))
    rx, ry = b.dt / b.dx, b.dt / b.dy
    d = h + e
    us, vs = u - b.g * rx * (east(e) - e), v - b.g * ry * (north(e) - e)
    if flags & ADVECTION:
        vb = 0.25 * (v + east(v) + south(v) + south(east(v)))
        ub = 0.25 * (u + west(u) + north(u) + north(west(u)))
        us = us - (torch.where(u > 0, u * (u - west(u)), u * (east(u) - u)) * rx
                   + torch.where(vb > 0, vb * (u - south(u)), vb * (north(u) - u)) * ry)
        vs = vs - (torch.where(ub > 0, ub * (v - west(v)), ub * (east(v) - v)) * rx
                   + torch.where(v > 0, v * (v - south(v)), v * (north(v) - v)) * ry)
    if flags & FRICTION:
        us = us / (1.0 + b.dt * CD * u.abs() / (0.5 * (d + east(d))))
        vs = vs / (1.0 + b.dt * CD * v.abs() / (0.5 * (d + north(d))))
    us, vs = torch.where(wx, us, 0.0), torch.where(wy, vs, 0.0)
    fx, fy = us * torch.where(us > 0, d, east(d)), vs * torch.where(vs > 0, d, north(d))
    es = torch.where(w, e - rx * (fx - west(fx)) - ry * (fy - south(fy)), 0.0)
    if flags & FILTER_UV:
        return _filtered(es, w, b.eps), _filtered(us, wx, b.eps), _filtered(vs, wy, b.eps)
    return _filtered(es, w, b.eps), us, vs


def _exact_basin(b):
    w = b.mask != 0
    return ([t.double() for t in (b.eta, b.u, b.v)], torch.where(w, b.H.double(), 0.0), w, w & _shift(w, 0, 1),
            w & _shift(w, 1, 0))


def _exact_steps(b, steps, flags=0):
    state, h, w, wx, wy = _exact_basin(b)
    for _ in range(steps):
        state = _exact_step(*state, h, w, wx, wy, b, flags)
    return state


def _taps(x):
    """The nine shifted copies of x [n, h, w, c], zero outside, as [n h w, c] matrices."""
    n, h, w, c = x.shape
    p = torch.zeros((n, h + 2, w + 2, c), dtype=x.dtype, device=x.device)
    p[:, 1:-1, 1:-1] = x
    for ky in range(3):
        for kx in range(3):
            yield p[:, ky:ky + h, kx:kx + w].reshape(-1, c)


def _layers(net):
    """(BF16-rounded weight, its FP32 bias) of each layer in 64 bits."""
    return [(net.wk[layer].double(), net.weight(layer)[1].double()) for layer in range(4)]


def _conv(x, weight, bias):
    y = bias.repeat(x.shape[0] * x.shape[1] * x.shape[2], 1)
    for t, a in enumerate(_taps(x)):
        y.addmm_(a, weight[t].t())
    return y.reshape(*x.shape[:3], 32)


def _network(x, layers):
    """Outputs of every layer (after the ReLU in the first three) for x [n, h, w, 16]."""
    acts = []
    for layer, (weight, bias) in enumerate(layers):
        x = _conv(x, weight, bias)
        x = x.clamp(min=0.0) if layer < 3 else x
        acts.append(x)
    return acts


def _packed(eta, u, v, H, mask, noise=None):
    x = torch.stack([eta, u, v, H, (mask != 0).double()], dim=-1).double()
    x = (x - _cuda64(np.float32(IN_MEAN))) / _cuda64(np.float32(IN_STD))
    if noise is not None:
        x[..., :3] += noise
    return torch.cat([x, torch.zeros(*x.shape[:-1], 11, dtype=x.dtype, device=x.device)], dim=-1)


def _splitmix(seed, n):
    """U[i] in [-1, 1) of the counters 0..n-1 (SplitMix64), as the training noise is keyed."""
    def shr(z, k):
        return (z >> k) & ((1 << (64 - k)) - 1)

    def signed(c):
        return c - (1 << 64) if c >= 1 << 63 else c
    z = (torch.arange(1, n + 1, dtype=torch.int64, device="cuda") * signed(0x9E3779B97F4A7C15)) + signed(seed)
    z = (z ^ shr(z, 30)) * signed(0xBF58476D1CE4E5B9)
    z = (z ^ shr(z, 27)) * signed(0x94D049BB133111EB)
    z = z ^ shr(z, 31)
    return shr(z, 40).double() / 8388608.0 - 1.0


def _exact_corrected(case, seed):
    b = _basin(case["nx"], case["ny"], seed, scale=4.0)
    layers = _layers(_net(seed))
    (e, u, v), h, w, wx, wy = _exact_basin(b)
    for _ in range(case["rounds"]):
        out = _network(_packed(e, u, v, b.H.double(), b.mask)[None], layers)[3][0].permute(2, 0, 1)[:3]
        for _ in range(case["every"]):
            e, u, v = _exact_step(e, u, v, h, w, wx, wy, b, 0)
        scale = np.float32(T_STD).astype(np.float64)
        e, u, v = (x + torch.where(m, float(c) * o, 0.0) for x, m, c, o in zip((e, u, v), (w, wx, wy), scale, out))
    if case["every"] == 1:
        return {"eta": e, "u": u, "v": v}
    return {"eta": e, "u": u, "v": v, "out": out[None]}


def _exact_train(case, seed):
    n, nx, ny = case["batch"], case["nx"], case["ny"]
    ds, net = _dataset(case, seed), _net(seed)
    m, v = _moments(net, seed)
    layers = _layers(net)
    runs = torch.as_tensor(ds.run_of[:n]).cuda()
    noise = np.float64(np.float32(NOISE)) * torch.stack(
        [_splitmix((0x5EED << 32) ^ (j + 1), 3 * nx * ny).reshape(ny, nx, 3) for j in range(n)])
    mask = ds.mask[runs]
    x = _packed(*ds.inputs[:, :n], ds.H[runs], mask, noise)
    acts = _network(x, layers)
    w = mask != 0
    active = torch.stack([w, torch.zeros_like(w), torch.zeros_like(w)], dim=-1)
    active[:, :, :-1, 1] = w[:, :, :-1] & w[:, :, 1:]
    active[:, :-1, :, 2] = w[:, :-1] & w[:, 1:]
    target = ds.targets[:, :n].permute(1, 2, 3, 0).double() / _cuda64(np.float32(T_STD))
    r = torch.where(active, acts[3][..., :3] - target, 0.0)
    dy = torch.zeros_like(acts[3])
    dy[..., :3] = 2.0 * r / float(active.sum())
    grad = torch.zeros(net.n_params, dtype=torch.float64, device="cuda")
    for layer in (3, 2, 1, 0):
        x_in = acts[layer - 1] if layer else x
        w0, b0 = net.offsets[layer]
        flat = dy.reshape(-1, 32)
        grad[w0:b0] = torch.stack([flat.t() @ a for a in _taps(x_in)]).reshape(-1)
        grad[b0:b0 + 32] = flat.sum(0)
        if layer:
            weight = layers[layer][0]
            dx = torch.zeros_like(x_in).reshape(-1, 32)
            for t, a in enumerate(_taps(dy)):  # a: dy at p + off_t, which x[p] reached through tap 8 - t
                dx.addmm_(a, weight[8 - t])
            dy = dx.reshape(x_in.shape) * (x_in > 0)
    theta, t = net.theta.double(), 101
    m = 0.9 * m.double() + 0.1 * grad
    v = 0.999 * v.double() + 0.001 * grad ** 2
    theta = theta - LR * (m / (1 - 0.9 ** t)) / ((v / (1 - 0.999 ** t)).sqrt() + 1e-8)
    return {"loss": r.square().sum().reshape(1), "grad": grad, "theta": theta, "m": m, "v": v}


def _blocks(a):
    ny, nx = a.shape
    return a.reshape(ny // 4, 4, nx // 4, 4)


def _exact_restrict(state, H, w):
    e, u, v = state
    n = _blocks(w.double()).sum((1, 3))
    wc = n >= 8
    mean = lambda a: _blocks(torch.where(w, a, 0.0)).sum((1, 3)) / n.clamp(min=1.0)  # noqa: E731
    return (torch.where(wc, mean(e), 0.0), torch.where(wc & _shift(wc, 0, 1), _blocks(u)[:, :, :, 3].mean(1), 0.0),
            torch.where(wc & _shift(wc, 1, 0), _blocks(v)[:, 3].mean(2), 0.0), mean(H), wc)


def _exact_judge(case, seed):
    b = _basin(case["nx"], case["ny"], seed, border=4)
    start, H = [t.double() for t in (b.eta, b.u, b.v)], b.H.double()
    w = b.mask != 0
    ce, cu, cv, ch, cw = _exact_restrict(start, H, w)
    c = SimpleNamespace(dx=4 * b.dx, dy=4 * b.dy, g=b.g, dt=4 * b.dt, eps=b.eps, H=ch, mask=cw, eta=ce, u=cu, v=cv)
    ce = _exact_steps(c, 2)[0]
    e, u, v, h, wc = _exact_restrict(_exact_steps(b, 8), H, w)
    rmse = ((torch.where(wc, ce - e, 0.0).square().sum() / wc.sum()).sqrt()).item()
    return {"eta": e, "u": u, "v": v, "H": h, "mask": None, "rmse": rmse}


def _exact_sor(case, seed):
    p, f = (t.double() for t in _poisson(case, seed))
    cx, cy, cz, omega = 1.0 / 16.0, 1.0 / 16.0, 1.0 / 4.0, 1.7
    diag = 2.0 * (cx + cy + cz)
    k, j, i = (torch.arange(1, n - 1, device="cuda") for n in p.shape)
    black = ((k[:, None, None] + j[None, :, None] + i[None, None, :]) & 1).bool()
    inner = p[1:-1, 1:-1, 1:-1]
    fi = f[1:-1, 1:-1, 1:-1]

    def neighbours():
        return (cx * (p[1:-1, 1:-1, 2:] + p[1:-1, 1:-1, :-2]) + cy * (p[1:-1, 2:, 1:-1] + p[1:-1, :-2, 1:-1])
                + cz * (p[2:, 1:-1, 1:-1] + p[:-2, 1:-1, 1:-1]))
    top, total = [], []
    for n in range(case["iters"] + 1):
        r = fi - (neighbours() - diag * inner)
        top.append(r.abs().max())
        total.append(r.square().sum())
        if n == case["iters"]:
            break
        for colour in (~black, black):
            gs = (neighbours() - fi) / diag
            inner += torch.where(colour, omega * (gs - inner), 0.0)
    return {"p": p, "max_abs_r": torch.stack(top), "sum_r2": torch.stack(total)}


def exact(case, seed):
    kind = case["kind"]
    if kind == "step":
        if case["flags"] & WETDRY:
            return None  # its decisions may fall either way within rounding, and the states then part
        b = _basin(case["nx"], case["ny"], seed)
        return dict(zip(("eta", "u", "v"), _exact_steps(b, case["steps"], case["flags"])))
    if kind == "ensemble":
        states = [_exact_steps(b, case["steps"]) for b in _members(case, seed)]
        return {name: torch.cat([st[f].reshape(-1) for st in states]) for f, name in enumerate(("eta", "u", "v"))}
    return {"corrected": _exact_corrected, "train": _exact_train, "judge": _exact_judge,
            "sor": _exact_sor}[kind](case, seed)
