"""The reverse step's lane layout: widths at which the outlet's feeding
column would begin a wavefront (nx - 1 a multiple of 64, where the lanes are
shifted by one), their neighbours, and the narrowest lattice, whose one
interior column feeds both boundaries.  FP64 gradient against the oracle's
exact discrete gradient; the tolerance is that of the other FP64 adjoint
tests (rounding of 1e-16 over 12 steps, amplified by the gradient's spread
over the cells)."""
import pytest
import torch

import workloads as W
from oracle import adjoint2d as A
from oracle import lbm2d as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("options", [{}, dict(pressure_inlet=True, p_in=2e-4, p_out=0.0, sigma_energy=True,
                                              buoyancy=(1e-7, -2e-7), heat_physical=True)], ids=["plain", "options"])
@pytest.mark.parametrize("nx", [3, 4, 64, 65, 66, 128, 129, 257])
def test_gradient_at_lane_boundaries(nx, options):
    from paper_2103_01444_amd import lbm
    ny, nsteps, every = 9, 12, 5
    w = W.adjoint2d(nx, ny)
    w.update(ny_channel=4, ny_gdl=4, ny_cl=1, Re=2.0, V_op=0.45, precision=64, **options)
    phi = torch.as_tensor(W.porosity_field(w), dtype=torch.float64)
    g, p = L.geometry_from_workload(w), L.Params.from_workload(w)
    m = L.Model(g, p, phi=phi)
    fields = [phi, m.inv_k.detach().clone(), m.d_eff.detach().clone()]
    sim = lbm.Cathode.from_workload(w, phi=phi, independent_fields=1)
    J = sim.forward_checkpointed(nsteps, every)
    out = sim.backward(1.0)
    Jo, gphi, gk, gd = A.gradient(g, p, *fields, nsteps=nsteps, every=every)
    assert abs(J / float(Jo) - 1) < 1e-12
    for name, ref in (("phi", gphi), ("inv_k", gk), ("d_eff", gd)):
        ref = ref[4:]
        err = float((out[name].cpu()[4:] - ref).abs().max() / ref.abs().max().clamp_min(1e-300))
        print(f"nx {nx} d/d{name}: rel err {err:.2e}", flush=True)
        assert err < 1e-9, (name, err)


def _bits(t):
    return t.contiguous().view(torch.int64 if t.dtype == torch.float64 else torch.int32)


@pytest.mark.parametrize("precision", [32, 64])
@pytest.mark.parametrize("shape", [(3, 3), (59, 4), (60, 5), (61, 6), (62, 7), (121, 12), (122, 13), (181, 3),
                                   (2185, 60), (2186, 61), (541, 243)], ids=lambda s: f"{s[0]}x{s[1]}")
def test_reverse_pairs_equal_single_reverse_steps(shape, precision):
    """Two reverse steps per launch at the edges of their tiles (60 columns;
    two rows below 2^17 nodes, six above) against a checkpoint at every step,
    whose segments are swept one step at a time: the same gradient bits."""
    from paper_2103_01444_amd import lbm
    nx, ny = shape
    ch = max(1, ny // 2)
    w = W.adjoint2d(64, 16)
    w.update(nx=nx, ny=ny, ny_channel=ch, ny_gdl=ny - ch - 1, ny_cl=1, Re=0.5, V_op=0.45, precision=precision)
    phi = torch.as_tensor(W.porosity_field(w))
    sims = [lbm.Cathode.from_workload(w, phi=phi, independent_fields=1) for _ in range(2)]
    J = [s.forward_checkpointed(13, every) for s, every in zip(sims, (5, 1))]
    assert J[0] == J[1]
    a, b = (s.backward(1.0, permeability=False) for s in sims)
    for name in ("inv_k", "phi", "d_eff"):
        assert bool(torch.isfinite(a[name]).all()), name
        assert torch.equal(_bits(a[name]), _bits(b[name])), name
