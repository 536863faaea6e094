"""The checkpointed forward run takes pairs or single steps by the lattice's
size, cached or streaming ones by its state's: the states and gradients are
the same bits whichever form the segments' lengths and the replay choose."""

import pytest
import torch

import workloads as W
import paper_2103_01444_amd.lbm as lbm

pytestmark = pytest.mark.gpu

# below and at the 2^17 nodes from which a chain alone takes single steps, a
# state below and above 40 MB, one above 192 MB (one step's own rule)
SHAPES = [(512, 255, 32), (512, 256, 32), (515, 259, 64), (1031, 523, 32), (1031, 523, 64), (3001, 900, 32)]


def _sim(nx, ny, bits, flags):
    w = W.cathode2d_scaled(nx, ny, bits)
    return lbm.Cathode.from_workload(w, phi=W.porosity_field(w), independent_fields=1, flags=flags)


@pytest.mark.parametrize("flags", [0, 1])
@pytest.mark.parametrize("nx,ny,bits", SHAPES)
def test_states_and_gradients_of_one_segment_and_many(nx, ny, bits, flags):
    steps = 7
    ref = _sim(nx, ny, bits, flags)
    for _ in range(steps):
        ref.step(1)
    want = ref.populations()
    ref.close()
    grads = []
    sim = _sim(nx, ny, bits, flags)
    for every in (steps, 4, 3, 1):
        sim.forward_checkpointed(steps, every)
        assert torch.equal(sim.populations(), want), every
        grads.append(sim.backward())
    for g in grads[1:]:
        for name, v in grads[0].items():
            assert torch.equal(g[name], v), name
    assert all(bool(torch.isfinite(v).all()) for v in grads[0].values())
    assert float(grads[0]["phi"].abs().max()) > 0  # the flow has not reached the layers yet
    sim.close()
