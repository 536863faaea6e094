"""Rounding of the FP32 reverse sweep by itself: the GPU's FP32 gradient
against the 64-bit adjoint along the same FP32 trajectory (every state the
GPU's, every step's transposed Jacobian the FP64 oracle's).

Tolerance, 2-norm of each gradient: the reaction's rates and sensitivities
carry ten roundings that all cells share, and a step's own rounding adds like
the root of the steps: (10 + sqrt(steps)) 2^-24."""
import math

import pytest
import torch

import workloads as W
from oracle import lbm2d as L
from oracle import lbm3d as L3

pytestmark = pytest.mark.gpu
DT = torch.float64
CASES = {
    "2d": dict(shape=(42, 224), steps=106),
    "2d_options": dict(shape=(48, 67), steps=79,
                       opts=dict(pressure_inlet=True, p_in=4e-4, p_out=1e-4, butler_volmer=True, buoyancy=(1e-7, -2e-7),
                                 sigma_energy=True, heat_physical=True)),
    "3d": dict(shape=(30, 24, 48), steps=24),
}


def _case(name):
    c = CASES[name]
    n = c["shape"][0]
    layers = (n // 2, n - n // 2 - max(1, n // 20), max(1, n // 20))
    if len(c["shape"]) == 2:
        ny, nx = c["shape"]
        w = W.adjoint2d(nx, ny)
        w.update(ny_channel=layers[0], ny_gdl=layers[1], ny_cl=layers[2], Re=0.2 * layers[0], V_op=0.55,
                 **c.get("opts", {}))
        return w, L.geometry_from_workload(w), L.Params.from_workload(w), L.Model, c["steps"]
    nz, ny, nx = c["shape"]
    w = W.cathode3d_scaled(nx, ny, nz, precision=32, nz_channel=layers[0], nz_gdl=layers[1], nz_cl=layers[2],
                           Re=0.2 * layers[0], dp_lat=8.0)
    return w, L3.Geometry3D(nx, ny, nz, *layers), L3.params_from_workload(w), L3.Model3D, c["steps"]


@pytest.mark.parametrize("name", list(CASES))
def test_fp32_reverse_sweep_against_its_own_trajectory(name):
    from paper_2103_01444_amd import lbm
    w, geo, prm, model, steps = _case(name)
    gen = torch.Generator().manual_seed(3)
    phi = (0.4 + 0.4 * torch.rand(CASES[name]["shape"], generator=gen, dtype=DT)).float()
    phi[:CASES[name]["shape"][0] // 2] = 1.0
    m = model(geo, prm, phi=phi.double())
    fields = [phi, m.inv_k.detach().float(), m.d_eff.detach().float()]
    cls = lbm.Cathode if len(phi.shape) == 2 else lbm.Cathode3D
    sim = cls.from_workload(dict(w, precision=32), phi=fields[0], inv_k=fields[1], d_eff=fields[2],
                            independent_fields=1)
    states = [sim.populations().double().cpu()]
    for _ in range(steps):
        sim.step(1)
        states.append(sim.populations().double().cpu())

    leaves = [a.double().requires_grad_(True) for a in fields]
    m = model(geo, prm, phi=leaves[0], inv_k=leaves[1], d_eff=leaves[2])
    total = [torch.zeros_like(a) for a in leaves]

    def vjp(out, state, lam=None):
        r = torch.autograd.grad(out, ([] if state is None else [state]) + leaves, grad_outputs=lam, allow_unused=True,
                                retain_graph=True)
        for t, g in zip(total, r[-3:]):
            if g is not None:
                t += g
        return r[0]

    s = states[-1].requires_grad_(True)
    lam = vjp(m.observables(s)["current_density"], s)
    for n in range(steps - 1, -1, -1):
        s = states[n].requires_grad_(True)
        lam = vjp(m.step(s), s, lam)
    vjp(m.initial_state(), None, lam)

    sim.forward_checkpointed(steps, 17)
    g = sim.backward(1.0, permeability=False)
    tol = (10 + math.sqrt(steps)) * 2.0 ** -24
    for key, ref in zip(("phi", "inv_k", "d_eff"), total):
        err = float((g[key].double().cpu() - ref).norm() / ref.norm())
        print(f"{name} d/d{key}: {err:.2e} (tolerance {tol:.2e})", flush=True)
        assert err < tol, key
