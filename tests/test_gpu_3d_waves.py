"""The 3D step and reverse step at the edges of their wavefronts (64 nodes of
one row each, shifted by one lane in the reverse step where nx - 1 is a
multiple of 64): FP64 fields of a run and its gradient against the oracle, at
the narrowest lattice and on both sides of those widths.  Tolerances as in
the other FP64 3D tests (rounding over a few steps)."""
import pytest
import torch

import workloads as W
from oracle import adjoint3d as A3
from oracle import lbm3d as L3

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx", [3, 4, 63, 64, 65, 66, 129])
def test_step_and_gradient_at_wavefront_edges(nx):
    from paper_2103_01444_amd import lbm
    ny, nz, nsteps, every = 3, 6, 11, 4
    w = W.cathode3d_scaled(8, ny, nz, precision=64, nz_channel=3, nz_gdl=2, nz_cl=1, Re=0.8, V_op=0.45,
                           sphere_radius=1.5, filter_box=3)
    w["nx"] = nx
    phi = torch.ones(nz, ny, nx, dtype=torch.float64)
    phi[3:] = 0.4 + 0.4 * torch.rand(nz - 3, ny, nx, dtype=torch.float64, generator=torch.Generator().manual_seed(nx))
    g, p = L3.geometry_from_workload(w), L3.params_from_workload(w)
    m = L3.Model3D(g, p, phi=phi)
    fields = [phi, m.inv_k.detach().clone(), m.d_eff.detach().clone()]
    sim = lbm.Cathode3D.from_workload(w, phi=fields[0], inv_k=fields[1], d_eff=fields[2])
    J = sim.forward_checkpointed(nsteps, every)
    got = sim.fields()
    m = L3.Model3D(g, p, phi=fields[0], inv_k=fields[1], d_eff=fields[2])
    ref = m.fields(m.run(m.initial_state(), nsteps))
    u = max(float(ref[k].abs().max()) for k in ("ux", "uy", "uz"))
    for name in ("ux", "uy", "uz", "T", "c"):
        scale = u if name.startswith("u") else float(ref[name].abs().max())
        assert float((got[name].cpu() - ref[name]).abs().max()) / scale < 1e-12, name
    out = sim.backward(1.0)
    Jo, gphi, gk, gd = A3.gradient(g, p, *fields, nsteps=nsteps, every=every)
    assert abs(J / float(Jo) - 1) < 1e-12
    for name, want in (("phi", gphi), ("inv_k", gk), ("d_eff", gd)):
        want = want[3:]
        err = float((out[name].cpu()[3:] - want).abs().max() / want.abs().max().clamp_min(1e-300))
        print(f"nx {nx} d/d{name}: rel err {err:.2e}", flush=True)
        assert err < 1e-9, (name, err)
