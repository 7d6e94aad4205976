"""A discharge behind a blocking capacitor whose first call has several steps (runs on
an MI355X): it gives what stepping one by one gives, bit for bit.  The load's field is
solved at the source voltage itself, the fields after it at the potential that follows
from the charges, so the first step has to take the potential of the field that is
there."""
import numpy as np
import pytest

import workloads as W
from test_gpu_fused import _same, pm  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


def _params(k, fp64, **kw):
    # the two formulas of the potential differ in the last bits for about half of all starts
    p = W.discharge([0.025, 0.04, 0.075, 0.031][k], [64, 129, 512, 33][k], [100.0, 300.0, 200.0, 77.7][k], 200, 1.0,
                    5000 + 7 * k, 1e15, seed=9 + k, case_id=k, fp64=fp64)
    p.update(phase_rad=0.1 * k, v2_volt=[0.0, 300.0, 200.0, 50.0][k], phase2_rad=[0.0, 0.0, 0.6, 0.9][k],
             cb_f_m2=[2e-8, 1e-7][k % 2])
    p.update(kw)
    return p


@pytest.mark.parametrize("fp64", [True, False])
@pytest.mark.parametrize("k", range(4))
def test_first_call_of_several_steps(pm, k, fp64):
    p = _params(k, fp64)
    a, b = pm.Case(p), pm.Case(p)
    for n in (26, 1, 3, 40):
        a.step(n)
        for _ in range(n):
            b.step(1)
        _same(a, b, n)
    # other particles: the field is solved anew, its reference charge kept
    for c in (a, b):
        st = c.get_particles(0)
        o = np.argsort(st["id"])[:4000]
        c.set_particles(0, {key: v[o] for key, v in st.items()})
    a.step(30)
    for _ in range(30):
        b.step(1)
    _same(a, b, "new particles")


@pytest.mark.parametrize("fp64", [True, False])
@pytest.mark.parametrize("k", range(4))
def test_captured_cycles_from_the_load(pm, k, fp64):
    p = _params(k, fp64, sort_interval=40, n_phase=10, flux_profiles=1)
    a, b = pm.Case(p), pm.Case(p)
    for turn in range(2):
        a.step_rf_cycles(1)
        for _ in range(200):
            b.step(1)
        _same(a, b, turn)


@pytest.mark.parametrize("fp64", [True, False])
@pytest.mark.parametrize("lanes", [1, 2])
def test_batch_members_with_circuits_and_phase_bins(pm, lanes, fp64):
    def members():
        return [pm.Case(_params(k, fp64, n_phase=7 if k % 2 else 0, cb_f_m2=0.0 if k == 2 else 2e-8)) for k in range(4)]
    a, b = members(), members()
    fused, plain = pm.Batch(a), pm.Batch(b)
    for x in (fused, plain):
        x.set_launch_shape(lanes=lanes, sort_interval=25)
    for n in (26, 1, 3):
        fused.step(n)
        for _ in range(n):
            plain.step(1)
        for k, (u, v) in enumerate(zip(a, b)):
            _same(u, v, (n, k))
    fused.close()
    plain.close()
