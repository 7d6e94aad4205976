"""Several steps of one call run in one launch each, a single step in two (runs on
an MI355X).  Both do the same arithmetic on the same random numbers, so a case
stepped by one call and a case stepped step by step agree bit for bit: particles,
charge, field and every diagnostic."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

SEGMENTS = (1, 2, 3, 26, 7)
CASES = {
    "fp64": dict(),
    "fp32": dict(fp64=False),
    "fp64_flux_phase": dict(n_phase=7, flux_profiles=1, n_cells=1024),
    "fp32_flux_phase": dict(fp64=False, n_phase=100, flux_profiles=1, n_cells=129),
    "circuit": dict(fp64=False, cb_f_m2=2e-8, v2_volt=50.0, phase2_rad=0.3, n_cells=65),
    "one_cell": dict(n_cells=1, sort_interval=7),
    "two_cells_fp32": dict(fp64=False, n_cells=2, flux_profiles=1),
    "one_electron": dict(np_e=1, np_i=0, sort_interval=0),
    "ragged": dict(fp64=False, np_e=2047, np_i=2049, n_cells=777, sort_interval=2),
    "sort_each_step": dict(sort_interval=1),
    "no_field": dict(fp64=False, flags=1),
    "no_gas": dict(p_pa=0.0),
    # more candidates in a pass than lanes, and births by the hundred per step
    "dense": dict(p_pa=300.0, te_ev=20.0, steps_per_cycle=2000, capacity_e=60_000, capacity_i=60_000),
    "dense_fp32": dict(fp64=False, p_pa=300.0, te_ev=20.0, steps_per_cycle=2000, capacity_e=60_000,
                       capacity_i=60_000),
    # more passes than workgroups
    "passes": dict(fp64=False, np_e=700_001, np_i=650_003, capacity_e=800_000, capacity_i=800_000, n_cells=128,
                   flux_profiles=1),
    "passes_fp64": dict(np_e=400_001, np_i=350_003, capacity_e=500_000, capacity_i=500_000, n_cells=512),
}


@pytest.fixture(scope="module")
def pm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1607_04069_amd as mod
    return mod


def _params(name, seed):
    kw = dict(CASES[name])
    p = W.discharge_small(seed=seed, fp64=kw.pop("fp64", True))
    p.update(kw)
    return p


def _same(a, b, label):
    for s in (0, 1):
        u, v = a.get_particles(s), b.get_particles(s)
        i, j = np.argsort(u["id"]), np.argsort(v["id"])
        for k in u:
            assert np.array_equal(u[k][i], v[k][j], equal_nan=k != "id"), (label, s, k)
    for read in ("get_fields", "sample_diagnostics"):
        u, v = getattr(a, read)(), getattr(b, read)()
        for k in u:
            assert np.array_equal(u[k], v[k], equal_nan=True), (label, read, k)
    for bin in range(0, a.p.get("n_phase", 0), 3):
        u, v = a.sample_phase(bin), b.sample_phase(bin)
        for k in u:
            assert np.array_equal(u[k], v[k], equal_nan=True), (label, "phase", bin, k)


@pytest.mark.parametrize("name", sorted(CASES))
def test_one_launch_steps_are_the_two_launch_steps(pm, name):
    p = _params(name, seed=5)
    a, b = pm.Case(p), pm.Case(p)
    for n in SEGMENTS:
        print(f"{name}: {n} steps", flush=True)
        a.step(n)
        for _ in range(n):
            b.step(1)
        _same(a, b, (name, n))
    a.close()
    b.close()


@pytest.mark.parametrize("fp64", [True, False])
def test_cycles_and_checkpoints(pm, fp64):
    """A captured RF period, replayed with the program's own work in between, and
    a state saved between calls."""
    p = W.discharge_small(seed=8, fp64=fp64)
    p.update(steps_per_cycle=60, n_phase=6, flux_profiles=1, sort_interval=25)
    a, b, c = pm.Case(p), pm.Case(p), pm.Case(p)
    for k in range(3):
        print(f"cycle {k}", flush=True)
        a.step_rf_cycles(1)
        for _ in range(60):
            b.step(1)
        _same(a, b, ("cycle", k))
        c.load_checkpoint(a.save_checkpoint())
        a.step(5)
        c.step(5)
        for _ in range(5):
            b.step(1)
        _same(a, b, ("after the cycle", k))
        _same(a, c, ("restored", k))


@pytest.mark.parametrize("fault", ["capacity", "nan"])
def test_failures_are_reported_alike(pm, fault):
    p = _params("dense_fp32", seed=6)
    if fault == "capacity":
        p.update(capacity_e=5003, capacity_i=5003)
    seen = []
    for by_one in (False, True):
        case = pm.Case(p)
        if fault == "nan":
            st = case.get_particles(0)
            st["ux"][17] = np.nan
            case.set_particles(0, st)
        for n in (1,) * 30 if by_one else (30,):
            case.step(n)
        with pytest.raises(pm.PicMccError) as e:
            case.sample_diagnostics()
        seen.append(str(e.value))
        case.close()
    assert seen[0] == seen[1], seen
