"""Two steps per launch at the edges of the kernel's tiles (16 x 8 nodes on
lattices of fewer than 2^17 nodes, 48 x 8 on larger ones and in the batch):
one node short of, at and past a multiple of the tile, so that the outlet
opens a tile, its feeding column closes one, and the last row or column is
alone; the narrowest lattices; both sides of the size where the tile
changes.  A run of n steps in one call against n calls of one step, bit for
bit, and a batch's two-step schedule against single lattices."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def _bits(t):
    return t.contiguous().view(torch.int64 if t.dtype == torch.float64 else torch.int32)


def _workload(nx, ny, precision):
    ch, cl = ny // 2, max(1, ny // 10)
    w = W.cathode2d_scaled(64, 40, precision=precision)
    w.update(nx=nx, ny=ny, ny_channel=ch, ny_gdl=ny - ch - cl, ny_cl=cl, Re=min(5.0, 0.2 * ch))
    return w


@pytest.mark.parametrize("precision", [32, 64])
@pytest.mark.parametrize("shape", [(3, 3), (4, 8), (15, 7), (16, 8), (17, 9), (18, 10), (33, 24), (47, 5),
                                   (2730, 48), (2731, 48), (2737, 49), (2736, 57), (193, 681), (194, 680)],
                         ids=lambda s: f"{s[0]}x{s[1]}")
def test_pairs_equal_single_steps(shape, precision):
    from paper_2103_01444_amd import lbm
    nx, ny = shape
    w = _workload(nx, ny, precision)
    phi = torch.as_tensor(W.porosity_field(w))
    a, b = [lbm.Cathode.from_workload(w, phi=phi, independent_fields=1) for _ in range(2)]
    pops = torch.from_numpy(W.random_populations(ny, nx, nx + ny))
    for s in (a, b):
        s.set_populations(pops)
    a.step(9)
    for _ in range(9):
        b.step(1)
    assert torch.equal(_bits(a.populations()), _bits(b.populations()))


@pytest.mark.parametrize("precision", [32, 64])
def test_batch_two_step_tiles(precision):
    """Sizes at the edges of the batch's tiles, an even and an odd count."""
    from paper_2103_01444_amd import lbm
    cases = [_workload(nx, ny, precision) for nx, ny in ((3, 3), (47, 7), (48, 8), (49, 9), (50, 17), (97, 3), (200, 40))]
    sw = lbm.BatchedSweep(cases)
    sw.set_schedule(64, 12, 0, 960)
    single = [lbm.Cathode.from_workload(w) for w in cases]
    for n in (6, 5):
        sw.step(n)
        for i, s in enumerate(single):
            s.step(n)
            assert torch.equal(_bits(sw.populations(i)), _bits(s.populations())), (i, n)
