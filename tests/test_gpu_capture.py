"""Steps recorded into a caller's HIP graph: each replay goes on from the state that the last one left
wherever the recorded calls make an even number of passes of the handle's own steps per pass."""
import pytest
import torch

from paper_1711_04471_amd import inputs
from paper_1711_04471_amd.sw2d import Sw2d, Sw2dBatch

pytestmark = pytest.mark.gpu


def _replays(make, record, state, replays=3):
    """Record the calls once, replay them, and compare every replay with eager calls."""
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream), make() as got, make() as want:
        record(got)
        record(want)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            record(got)
        busy = torch.zeros(1 << 16, device="cuda")
        for rep in range(replays):
            graph.replay()
            busy.add_(1.0)
            record(want)
            torch.cuda.synchronize()
            for x, y in zip(state(got), state(want)):
                assert torch.equal(x, y), rep


# (calls, the handle's steps per pass): an even number of such passes
EVEN = [((2,), 1), ((4,), 1), ((6,), 1), ((8,), 1), ((18,), 1), ((1, 1), 1), ((3, 5), 1), ((7, 2, 1), 1),
        ((4,), 3), ((6,), 3), ((18,), 3), ((3, 3), 3), ((2, 4, 1), 3), ((5,), 4), ((1, 5), 2)]


@pytest.mark.parametrize("calls,spp", EVEN)
def test_recorded_steps_go_on_at_every_replay(calls, spp):
    assert sum(-(-n // spp) for n in calls) % 2 == 0
    c = inputs.small_basin(150, 61, seed=5)

    def make():
        sim = Sw2d.from_case(c)
        sim.set_time_blocking(spp, rows=8)
        return sim

    _replays(make, lambda s: [s.step(n) for n in calls], lambda s: s.state())


@pytest.mark.parametrize("shape,flags", [((150, 61), 0), ((1500, 1501), 1), ((3001, 2900), 0), ((3001, 2900), 8)])
@pytest.mark.parametrize("n", [2, 6])
def test_recorded_steps_of_a_default_handle(n, shape, flags):
    """One to 4 steps per pass by the grid and the model, friction 2 past 2^21 cells."""
    make_case = inputs.shore_basin if flags == 8 else inputs.small_basin
    c = make_case(*shape, seed=sum(shape))
    _replays(lambda: Sw2d.from_case(c, flags=flags, cd=0.0025, hmin=0.0625), lambda s: s.step(n), lambda s: s.state())


@pytest.mark.parametrize("grid,launch", [(0, 50), (64, 50), (64, 7)])
@pytest.mark.parametrize("n,K", [(2, 1), (4, 1), (6, 1), (10, 1), (20, 1), (4, 2), (12, 2), (6, 3), (12, 3), (18, 3)])
def test_recorded_ensemble_steps_go_on_at_every_replay(n, K, grid, launch):
    """Without the library's own graph, a launch per pass or persistent launches."""
    assert n // K % 2 == 0
    cases = [inputs.small_basin(*s, seed=3) for s in ((64, 64), (200, 180))]

    def make():
        b = Sw2dBatch(cases)
        b.set_time_blocking(K)
        b.set_launch(launch, False, grid)
        return b

    _replays(make, lambda b: b.step(n), lambda b: [x for k in range(b.n) for x in b.state(k)])
