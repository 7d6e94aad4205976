"""Every atom ends once (runs on an MI355X): the atoms at the target, at the substrate
and in the gas are counted apart, so their sum checks the atoms' way through the
queue, in flights too large to trace in full and in the shards they fall into."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1607_04069_amd as mod
    return mod


# large flights: one lane an atom, runs taken from the queue; a fixed step with an event limit
@pytest.mark.parametrize("p_pa,n,kw", [(0.5, 10_000_000, {}), (5.0, 1_000_000, {}),
                                       (0.5, 600_001, dict(dt_s=1e-6, e_max=40, scatter=1))])
def test_counts_add_up_over_shards(pm, p_pa, n, kw):
    src, tp = W.sputter_transport(p_pa=p_pa, n_atoms=n)
    tp.update(kw)
    whole = pm.run_test_particles(src, tp)
    keys = ("n_substrate", "n_target", "n_unfinished", "events", "collisions")
    assert whole["n_substrate"] + whole["n_target"] + whole["n_unfinished"] == n
    assert whole["n_target"] > n // 10 and whole["n_substrate"] > n // 10
    # shards of every number of lanes an atom, and their traces
    cuts = [0, 1, 1000, 20_000, 80_003, 200_001, n]
    sums = dict.fromkeys(keys, 0)
    for a, b in zip(cuts, cuts[1:]):
        part = pm.run_test_particles(dict(src, first_atom=a, n_atoms=b - a), tp, trace=b - a < 130_000)
        assert part["n_substrate"] + part["n_target"] + part["n_unfinished"] == b - a
        if "trace" in part:
            assert part["n_target"] == int((part["trace"]["wall"] == 0).sum())
        for k in keys:
            sums[k] += part[k]
    assert sums == {k: whole[k] for k in keys}
