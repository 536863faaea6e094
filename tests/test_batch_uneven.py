"""Batches of very uneven lattices: scratch and launches are the sum over the
cases, not the largest case's times their number."""
import ctypes

import numpy as np
import pytest
import torch

import workloads as W


def _geometry(lbm, nx, ny, precision=32):
    ch, cl = ny // 2, max(1, ny // 20)
    return lbm.Geometry(nx, ny, ch, ny - ch - cl, cl, precision, 0)


@pytest.mark.parametrize("precision", [32, 64])
def test_workspace_is_the_sum_over_the_cases(precision):
    """CPU: the library's host code alone."""
    from paper_2103_01444_amd import lbm
    lib = lbm.load_library()

    def nbytes(sizes):
        g = (lbm.Geometry * len(sizes))(*[_geometry(lbm, nx, ny, precision) for nx, ny in sizes])
        return lib.lbm_batch_workspace_bytes(g, len(sizes))

    big, small = [(4096, 1024)], [(200, 40)] * 255
    apart = nbytes(big) + nbytes(small)
    assert 0 < nbytes(big + small) <= apart + (1 << 16)  # a few regions are rounded up once instead of twice


@pytest.mark.gpu
@pytest.mark.parametrize("fields", [False, True], ids=["layered", "fields"])
@pytest.mark.parametrize("sizes", [[(600, 300), (3, 3), (257, 5), (256, 4), (5, 90)], [(9, 3)] * 300 + [(300, 40)]],
                         ids=["mixed", "301 cases"])
def test_uneven_cases_equal_single_lattices(sizes, fields):
    from paper_2103_01444_amd import lbm
    cases = []
    for nx, ny in sizes:
        ch, cl = ny // 2, max(1, ny // 20)
        w = W.cathode2d_scaled(64, 40, precision=32)
        w.update(nx=nx, ny=ny, ny_channel=ch, ny_gdl=ny - ch - cl, ny_cl=cl, Re=min(5.0, 0.2 * ch))
        cases.append(w)
    phi = [torch.as_tensor(W.porosity_field(w)) if fields else None for w in cases]
    b = lbm.BatchedSweep(cases, fields=[dict(phi=p) for p in phi] if fields else None)
    picks = sorted({0, 1, 2, len(cases) // 2, len(cases) - 2, len(cases) - 1})
    single = {i: lbm.Cathode.from_workload(cases[i], **(dict(phi=phi[i], independent_fields=1) if fields else {}))
              for i in picks}
    for schedule in ((256, 1, 0, 0), (64, 12, 0, 960)):
        b.init_equilibrium()
        b.set_schedule(*schedule)
        for s in single.values():
            s.init_equilibrium()
        for n in (0, 1, 5):
            b.step(n)
            obs = b.observables()
            assert len(obs) == len(cases)
            for i, s in single.items():
                s.step(n)
                assert torch.equal(b.populations(i), s.populations()), (i, n)
                ref = s.observables()
                for key in obs[i]:
                    assert obs[i][key] == ref[key] or (np.isnan(obs[i][key]) and np.isnan(ref[key])), (i, n, key)
