"""Flights whose histograms fill a workgroup's LDS (runs on an MI355X): the energy and
time bins that fit are counted as with room to spare, and those that do not are
refused as before."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

LDS = 160 * 1024
OWN = 48            # bytes of the kernel's own sums and counters beside the histograms


@pytest.fixture(scope="module")
def pm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1607_04069_amd as mod
    return mod


# bytes left beside the histograms: too few for a sum per lane, just enough, plenty
@pytest.mark.parametrize("spare", [OWN, 1000, 2048, 2064, 2072, 40_000])
@pytest.mark.parametrize("kw", [{}, dict(n_xbins=0), dict(dt_s=1e-7, scatter=1)])
def test_histograms_up_to_the_lds(pm, spare, kw):
    src, tp = W.sputter_transport(p_pa=2.0, n_atoms=20_011)
    tp.update(kw)
    profiles = 32 * (tp["n_xbins"] + 1) if tp["n_xbins"] else 0
    bins = (LDS - spare - profiles) // 4 - 90
    # the bins' widths are those of the small run: what falls beyond its last bin falls into later ones here
    big = pm.run_test_particles(src, dict(tp, n_ebins=bins - 300, n_tbins=300))
    ref = pm.run_test_particles(src, dict(tp, n_tbins=300))
    n = tp["n_ebins"]
    assert np.array_equal(big["e_hist"][:n - 1], ref["e_hist"][:n - 1])
    assert big["e_hist"][n - 1:].sum() == ref["e_hist"][n - 1]
    for k in ref:
        if k != "e_hist":
            assert np.array_equal(big[k], ref[k]), k


def test_histograms_beyond_the_lds_are_refused(pm):
    src, tp = W.sputter_transport(p_pa=2.0, n_atoms=100)
    tp.update(n_xbins=0, n_ebins=LDS // 4, n_tbins=300)
    with pytest.raises(pm.PicMccError):
        pm.run_test_particles(src, tp)
