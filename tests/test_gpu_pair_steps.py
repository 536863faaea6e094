"""Pairs of steps (a run's last two or four steps, which store no state
between, and the checkpointed runs' chains) at the edges of their tiles: 16 x 8
nodes on lattices of fewer than 2^17 nodes, 48 x 8 on larger ones.  A call of
two or four steps against single steps, bit for bit: one node short of, at and
past a multiple of the tile, both sides of the size where the tile changes,
every material form, and the model options."""
import pytest
import torch

import workloads as W
from oracle import lbm2d as L

pytestmark = pytest.mark.gpu
OPTIONS = {
    "butler_volmer_heat": dict(butler_volmer=True, alpha_a=0.5, V_op=1.1, aj0_ref=1e5, heat_physical=True),
    "buoyancy_sigma": dict(buoyancy=(3e-7, -5e-7), sigma_energy=True, heat_physical=True),
    "pressure_inlet_outlet": dict(pressure_inlet=True, p_in=4e-4, p_out=1e-4),
    "no_cl": {},
    "thin_cl": dict(thin_cl=True, butler_volmer=True, alpha_a=0.5, V_op=1.1, aj0_ref=1e5, sigma_energy=True),
}


def _bits(t):
    return t.contiguous().view(torch.int64 if t.dtype == torch.float64 else torch.int32)


def _workload(nx, ny, precision, **over):
    ch, cl = ny // 2, max(1, ny // 10)
    w = W.cathode2d_scaled(64, 40, precision=precision)
    w.update(nx=nx, ny=ny, ny_channel=ch, ny_gdl=ny - ch - cl, ny_cl=cl, Re=min(5.0, 0.2 * ch), **over)
    return w


def _fields(w, mode):
    if mode == "layered":
        return {}
    phi = torch.as_tensor(W.porosity_field(w))
    if mode == "phi":
        return dict(phi=phi)
    m = L.Model(L.Geometry(w["nx"], w["ny"], w["ny_channel"], w["ny_gdl"], w["ny_cl"]), L.Params.from_workload(w),
                phi=phi)
    return dict(phi=phi, inv_k=m.inv_k.detach(), d_eff=m.d_eff.detach(), independent_fields=1)


def _check(w, mode, label):
    from paper_2103_01444_amd import lbm
    kw = _fields(w, mode)
    a, b = [lbm.Cathode.from_workload(w, **kw) for _ in range(2)]
    pops = torch.from_numpy(W.random_populations(w["ny"], w["nx"], w["nx"] + w["ny"]))
    for s in (a, b):
        s.set_populations(pops)
    for n in (2, 2, 4, 2):
        a.step(n)
        for _ in range(n):
            b.step(1)
        assert torch.equal(_bits(a.populations()), _bits(b.populations())), (label, n)
    assert a.step_count == b.step_count == 10


@pytest.mark.parametrize("precision", [32, 64])
@pytest.mark.parametrize("mode", ["layered", "phi", "full"])
@pytest.mark.parametrize("shape", [(3, 3), (15, 7), (16, 8), (17, 9), (18, 10), (33, 24), (47, 5), (2730, 48),
                                   (2731, 48), (2737, 49), (2736, 57), (193, 681), (194, 680), (1027, 865)],
                         ids=lambda s: f"{s[0]}x{s[1]}")
def test_pairs_equal_single_steps(shape, mode, precision):
    _check(_workload(*shape, precision), mode, f"{shape} {mode} fp{precision}")


@pytest.mark.parametrize("precision", [32, 64])
@pytest.mark.parametrize("shape", [(49, 17), (1025, 515)], ids=["49x17", "1025x515"])
@pytest.mark.parametrize("option", list(OPTIONS))
def test_pairs_equal_single_steps_with_options(option, shape, precision):
    w = _workload(*shape, precision, **OPTIONS[option])
    if option in ("no_cl", "thin_cl"):
        w.update(ny_gdl=w["ny_gdl"] + w["ny_cl"], ny_cl=0)
    _check(w, "full", f"{option} {shape} fp{precision}")
