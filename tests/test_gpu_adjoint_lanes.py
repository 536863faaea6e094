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
