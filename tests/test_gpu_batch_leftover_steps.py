"""The steps left over from the batch's three-step schedule: one or two of
them take no longer than three, and give the bits of single lattices."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def _time(batch, n, repeats=10):
    """Least of several timings of n steps, milliseconds."""
    best = float("inf")
    for _ in range(8):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(repeats):
            batch.step(n)
        e1.record()
        e1.synchronize()
        best = min(best, e0.elapsed_time(e1) / repeats)
    return best


@pytest.mark.parametrize("precision", [32, 64])
def test_leftover_steps_take_no_longer_than_three(precision):
    from paper_2103_01444_amd import lbm
    b = lbm.BatchedSweep([dict(w, precision=precision) for w in W.batched_cases()])
    b.set_schedule(64, 12, 0, 960)
    one, two, three = (_time(b, n) for n in (1, 2, 3))
    print(f"fp{precision}: {one * 1e3:.0f}, {two * 1e3:.0f}, {three * 1e3:.0f} us", flush=True)
    assert two < 1.05 * three
    assert one < 1.05 * three


@pytest.mark.parametrize("fields", [False, True], ids=["layered", "fields"])
@pytest.mark.parametrize("precision", [32, 64])
def test_every_remainder_equals_single_lattices(precision, fields):
    """Model options on, sizes at the edges of the tiles."""
    from paper_2103_01444_amd import lbm
    cases = []
    for nx, ny in ((3, 3), (26, 11), (27, 12), (28, 13), (55, 25), (200, 40)):
        ch, cl = ny // 2, max(1, ny // 10)
        w = W.cathode2d_scaled(64, 40, precision=precision)
        w.update(nx=nx, ny=ny, ny_channel=ch, ny_gdl=ny - ch - cl, ny_cl=cl, Re=min(5.0, 0.2 * ch),
                 buoyancy=(1e-7, -2e-7), sigma_energy=True, heat_physical=True, pressure_inlet=True, p_in=1e-4)
        cases.append(w)
    phi = [torch.as_tensor(W.porosity_field(w)) if fields else None for w in cases]
    b = lbm.BatchedSweep(cases, fields=[dict(phi=p) for p in phi] if fields else None)
    b.set_schedule(64, 12, 0, 960)
    single = [lbm.Cathode.from_workload(w, **(dict(phi=p, independent_fields=1) if fields else {}))
              for w, p in zip(cases, phi)]
    for n in range(1, 9):
        b.step(n)
        for i, s in enumerate(single):
            for _ in range(n):
                s.step(1)
            assert torch.equal(b.populations(i), s.populations()), (n, i)
