"""A batch case whose rows are too long for 32-bit lane offsets (64 rows of 19
interleaved planes reach 2^32 bytes at 441 000 nodes a row): the general
addressing, against the single lattice, bit for bit."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("schedule", [(256, 1, 0, 0), (64, 2, 0, 128), (64, 12, 0, 960), (64, 4, 1, 0)],
                         ids=["rows", "tiles", "threes", "persistent"])
@pytest.mark.parametrize("precision", [32, 64])
def test_wide_rows_equal_single_lattice(precision, schedule):
    from paper_2103_01444_amd import lbm
    w = W.cathode2d_scaled(64, 40, precision=precision)
    w.update(nx=450001, ny=5, ny_channel=2, ny_gdl=2, ny_cl=1, Re=0.4)
    b = lbm.BatchedSweep([w, dict(w, nx=33)])
    b.set_schedule(*schedule)
    s = lbm.Cathode.from_workload(w)
    for n in (1, 2, 3):
        b.step(n)
        s.step(n)
        assert torch.equal(b.populations(0), s.populations()), n
    assert b.observables()[0]["sum_c"] == s.observables()["sum_c"]
