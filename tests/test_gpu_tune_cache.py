"""Tuner: trials time each form in its own launches.  Cache entries belong to the kernels and the material form they were
timed on: an entry under an older key, or of the other form, is not used."""
import json

import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def _batch(fields=False):
    from paper_2103_01444_amd import lbm
    cases = W.batched_cases(3)
    f = [dict(phi=torch.full((w["ny"], w["nx"]), 0.7)) for w in cases] if fields else None
    return lbm.BatchedSweep(cases, fields=f), cases


def test_entry_of_other_kernels_is_not_used(tmp_path):
    """The key of the earliest format: architecture, precision and sizes."""
    b, cases = _batch()
    path = tmp_path / "tune.json"
    old = "gfx950|fp32|" + ",".join(f"{w['nx']}x{w['ny']}" for w in cases)
    path.write_text('{\n"%s": {"tile_x": 1024, "tile_y": 1, "persistent": 1, "block": 0, "ms_per_step": 1e-09}\n}\n' % old)
    r = b.autotune(trial_steps=3, cache_path=str(path))
    assert not r["cached"] and r["ms_per_step"] > 1e-6
    entries = json.loads(path.read_text())
    assert len(entries) == 2 and entries[old]["tile_x"] == 1024  # kept, and a new one beside it
    assert b.autotune(trial_steps=3, cache_path=str(path))["cached"]


def test_material_forms_have_entries_of_their_own(tmp_path):
    path = str(tmp_path / "tune.json")
    assert not _batch()[0].autotune(trial_steps=3, cache_path=path)["cached"]
    assert not _batch(fields=True)[0].autotune(trial_steps=3, cache_path=path)["cached"]
    assert _batch(fields=True)[0].autotune(trial_steps=3, cache_path=path)["cached"]
    assert _batch()[0].autotune(trial_steps=3, cache_path=path)["cached"]


@pytest.mark.parametrize("trial_steps", [1, 2, 4])
def test_short_trials_time_the_three_step_form(trial_steps):
    """A trial that is no multiple of three is timed in launches of three, as
    a run has them: on the 64-case sweep that form takes half of any other's
    time a step."""
    from paper_2103_01444_amd import lbm
    b = lbm.BatchedSweep(W.batched_cases())
    b.step(4)
    before = [b.populations(i).clone() for i in (0, 31, 63)]
    r = b.autotune(trial_steps=trial_steps)
    print(r, flush=True)
    assert r["block"] == 960
    assert b.step_count == 4
    for i, p in zip((0, 31, 63), before):
        assert torch.equal(b.populations(i), p)
