"""The atom flight gives an atom one lane in a large launch and up to 64 in a small
one (runs on an MI355X).  An atom's arithmetic does not depend on that: the same
atoms agree bit for bit between launches of every size, and with the oracle."""
import numpy as np
import pytest

from oracle import tpm as T
import workloads as W

pytestmark = pytest.mark.gpu

# atoms of the launch with one lane per atom: above 64 (128 with a fixed step) x 4096
N_ONE_LANE = 530_000
CASES = {
    "vhs": dict(p_pa=2.0),
    "m1_substrate": dict(p_pa=2.0, scatter=1, electrode=1),
    "fixed_m1": dict(p_pa=5.0, scatter=1, dt_s=1e-7),
    "fixed_box": dict(p_pa=5.0, mode=1, dt_s=1e-7, e_max=70),
    "box": dict(p_pa=5.0, mode=1, e_max=37),
    "event_limit": dict(p_pa=5.0, e_max=17),
    "no_gas": dict(p_pa=0.0),
    "no_profiles": dict(p_pa=2.0, n_xbins=0),
    "one_cell": dict(p_pa=2.0, n_xbins=1),
}


@pytest.fixture(scope="module")
def pm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1607_04069_amd as mod
    return mod


def _inputs(n_atoms, first_atom=0, **kw):
    src, tp = W.sputter_transport(p_pa=kw["p_pa"], n_atoms=n_atoms, mode=kw.get("mode", 0))
    src.update(first_atom=first_atom, electrode=kw.get("electrode", 0))
    tp.update({k: v for k, v in kw.items() if k in ("scatter", "dt_s", "e_max", "n_xbins")})
    return src, tp


@pytest.mark.parametrize("name", list(CASES))
def test_lanes_per_atom_do_not_change_an_atom(pm, name):
    kw = CASES[name]
    big = pm.run_test_particles(*_inputs(N_ONE_LANE, **kw), trace=True)["trace"]
    # 64 or 16 lanes per atom; eight, four, two; runs that end inside a wavefront
    for n, first in ((1, 5), (63, 100), (4097, 1000), (16_385, 7), (66_000, 30_001), (140_003, 389_997)):
        small = pm.run_test_particles(*_inputs(n, first, **kw), trace=True)
        for k, v in small["trace"].items():
            assert np.array_equal(v, big[k][first:first + n], equal_nan=v.dtype.kind == "f"), (name, n, k)
        assert small["events"] == int(small["trace"]["events"].astype(np.int64).sum())
        assert small["n_substrate"] == int((small["trace"]["wall"] == 1).sum())
        assert small["n_target"] == int((small["trace"]["wall"] == 0).sum())


@pytest.mark.parametrize("name,n", [("vhs", 300), ("vhs", 9000), ("m1_substrate", 2500), ("fixed_m1", 700),
                                    ("event_limit", 5000)])
def test_wide_flights_match_the_oracle(pm, name, n):
    """Per atom the wall and event count for all but 1 % (FP32 against FP64 flips a
    decision within ~1e-6 of its threshold), tallies and profiles within 3 %."""
    src, tp = _inputs(n, **CASES[name])
    g = pm.run_test_particles(src, tp, trace=True)
    o = T.run(src, tp, trace=True)
    same = (g["trace"]["wall"] == o["trace"]["wall"]) & (g["trace"]["events"].astype(np.int64) == o["trace"]["events"])
    assert 1 - same.mean() <= 0.01
    assert abs(g["collisions"] - o["collisions"]) <= 0.03 * o["collisions"]
    assert abs(g["time_s"].sum() / o["time_s"].sum() - 1) <= 0.03
    assert abs(g["e_sum_target"] + g["e_sum_substrate"] - o["e_sum_target"] - o["e_sum_substrate"]) <= \
        0.03 * (o["e_sum_target"] + o["e_sum_substrate"])
