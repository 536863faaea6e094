"""Steps captured into a HIP graph: a graph of an even number of steps
advances the state at every replay, as a run of that many steps does, whatever
launches the steps are grouped into."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu
COUNTS = (2, 4, 6, 8, 10, 14, 20)


def _replays(make, states, n):
    """Capture n steps once, replay thrice with eager work between, and check
    each replay against an eager run."""
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        sim, ref = make(), make()
        sim.step(2)  # loads the kernels
        sim.init_equilibrium()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            sim.step(n)
        ref.init_equilibrium()
        for replay in range(3):
            graph.replay()
            ref.step(n)
            torch.cuda.synchronize()
            for i, (a, b) in enumerate(zip(states(sim), states(ref))):
                assert torch.equal(a, b), (n, replay, i)
            torch.ones(1000, device="cuda").cumsum(0)


def _w(nx, ny, precision):
    ch, cl = ny // 2, max(1, ny // 10)
    w = W.cathode2d_scaled(64, 40, precision=precision)
    w.update(nx=nx, ny=ny, ny_channel=ch, ny_gdl=ny - ch - cl, ny_cl=cl, Re=min(5.0, 0.2 * ch))
    return w


@pytest.mark.parametrize("n", COUNTS)
@pytest.mark.parametrize("shape", [(200, 40), (700, 300)], ids=["200x40", "700x300"])
def test_lattice(shape, n):
    from paper_2103_01444_amd import lbm
    _replays(lambda: lbm.Cathode.from_workload(_w(*shape, 32)), lambda s: [s.populations()], n)


@pytest.mark.parametrize("n", COUNTS)
@pytest.mark.parametrize("schedule", [(256, 1, 0, 0), (64, 12, 0, 960)], ids=["rows", "threes"])
def test_batch(schedule, n):
    from paper_2103_01444_amd import lbm

    def make():
        b = lbm.BatchedSweep([_w(200, 40, 32), _w(65, 33, 32)])
        b.set_schedule(*schedule)
        return b
    _replays(make, lambda b: [b.populations(0), b.populations(1)], n)


@pytest.mark.parametrize("n", (2, 4))
def test_lattice_3d(n):
    from paper_2103_01444_amd import lbm
    w = W.cathode3d_scaled(40, 12, 16, precision=32, dp_lat=0.0, Da_gdl=1e-3, Re=1.0)
    _replays(lambda: lbm.Cathode3D.from_workload(w), lambda s: [s.populations()], n)
