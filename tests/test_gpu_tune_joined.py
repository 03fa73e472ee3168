"""The joined form of the ADR levels as a candidate of the tuner (stored as no entry): it is timed
wherever it applies and the fastest timing of each level is what is stored; a context tuned
before it has a phase, and one with a cache file from before the form was a candidate, do
not lose it; where levels cannot be joined, a form is stored for each.
"""
import json
import re

import numpy as np
import pytest
import torch

import helm_inputs as hi
from gpu_util import TOL, assert_close, rand_grid, rounded, to_dev
from oracle.cycle import Problem, cycle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def case():
    return hi.make_problem(256, 160.0, 5, seed=4, medium="grf", phase="fmm", damping_cells=16)


def _context(c, phase=True, **kw):
    from paper_2404_02493_amd import Helmholtz

    H = Helmholtz(c.velocity, c.k, levels=c.levels, precision="c64", damping_cells=16, **kw)
    if phase:
        H.set_phase(c.phi)
    return H


def _joined(H, c):
    """Whether a cycle's level-2 steps run joined."""
    g = to_dev(rounded(torch.as_tensor(c.g), H.cdtype), H.cdtype)
    H.profile_begin()
    H.cycle(g, torch.zeros_like(g))
    return any("k_fuse_step" in k["name"] for k in H.profile_end()["kernels"])


def _forms(res, level):
    """{stored form: ms} of a level's timings (0: joined)."""
    names = {"joined": 0, "tile16": 1, "tile32": 2}
    out = {}
    for key, ms in res["timings_ms"].items():
        m = re.fullmatch(rf"sstep_l{level}_(\w+)", key)
        if m:
            out[names[m[1]] if m[1] in names else int(m[1])] = ms
    return out


def _is_fastest(form, forms):
    return forms[form] <= min(forms.values()) + 1e-5  # printed to 1e-5 ms


def test_fastest_timing_is_stored(case):
    H = _context(case)
    res = H.tune()
    timed = {l: _forms(res, l) for l in (2, 3, 4)}
    print(json.dumps(res["sstep_rows"]), {l: (min(timed[l].values()), timed[l].get(0)) for l in (2, 3)}, flush=True)
    assert 0 in timed[2] and 0 in timed[3] and not timed[4]  # level 4 of 64^2 or less: one workgroup alone
    assert _is_fastest(res["sstep_rows"].get("2", 0), timed[2])
    if "2" in res["sstep_rows"]:
        assert _is_fastest(res["sstep_rows"].get("3", 0), timed[3])
    else:  # joined steps take every level below along
        assert res["sstep_rows"] == {}
    H.close()


def test_tuned_before_the_phase(case):
    """Nothing to time the joined steps with: level 2 keeps its default, and the context stays
    joined if its lower levels do; parity as for every tuned context."""
    H = _context(case, phase=False)
    res = H.tune()
    H.set_phase(case.phi)
    assert "sstep_l2_joined" not in res["timings_ms"]
    if "3" not in res["sstep_rows"]:
        assert "2" not in res["sstep_rows"] and _joined(H, case)
    P = Problem(case.velocity, case.k, case.levels, damping_cells=16, phi=case.phi)
    H.set_weights(P.weights.numpy())
    u = rounded(rand_grid(np.random.default_rng(2), 256), H.cdtype)
    g = rounded(torch.as_tensor(case.g), H.cdtype)
    ud = to_dev(u, H.cdtype)
    H.cycle(to_dev(g, H.cdtype), ud)
    assert_close(ud, cycle(P, g, u), TOL["c64"], "cycle")
    H.close()


def test_old_cache_is_measured_again(case, tmp_path):
    """A cache file written when the joined form was no candidate does not bar it."""
    H = _context(case)
    old = re.sub(r"\|v\d+$", "|v4", H.tuning_key())
    path = tmp_path / "tune.json"
    path.write_text(json.dumps({old: {"sstep_rows": {"2": 1, "3": 1}, "fgmres_blocks": 512}}))
    res = H.tune(cache=str(path))
    assert "sstep_l2_joined" in res["timings_ms"]
    assert json.loads(path.read_text())[H.tuning_key()] == res
    H.close()


def test_levels_that_cannot_join_get_a_form(case):
    H = _context(case, gmres_m=2, tail_n=0)
    res = H.tune()
    assert set(res["sstep_rows"]) == {"2", "3", "4"}
    assert not any(k.endswith("_joined") for k in res["timings_ms"])
    for l in (2, 3, 4):
        assert _is_fastest(res["sstep_rows"][str(l)], _forms(res, l))
    assert not _joined(H, case)
    H.close()
