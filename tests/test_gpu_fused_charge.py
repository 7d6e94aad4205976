"""Particles a rounding below a cell edge, where a charge share in units of 2^-32
particle is a whole particle (runs on an MI355X): several steps of one call put it on
the same node as single steps and the oracle do."""
import numpy as np
import pytest

import workloads as W
from oracle import pic as P
from test_gpu_fused import _same, pm  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu

N = 33


def _positions(real, rng):
    """A wavefront's worth in one cell, then every cell's upper edge, then anything."""
    edge = np.arange(1, N + 1)
    below = np.nextafter(edge.astype(real), real(0)).astype(np.float64)
    if real is np.float64:
        below = np.concatenate([below, edge - 1e-12, edge - 2.0 ** -33, edge - 2.0 ** -34])
    return np.concatenate([np.full(1024, np.nextafter(real(10), real(0))), np.tile(below, 8),
                           rng.uniform(0, N, 777).astype(real)]).astype(np.float64)


def _case(pm, fp64, mode):
    # no voltage, no self field, no gas: the particles stay where they are put
    p = W.discharge_small(seed=3, fp64=fp64)
    p.update(n_cells=N, v0_volt=0.0, p_pa=0.0, flags=P.NO_SELF_FIELD, sort_interval=0, capacity_e=8000,
             capacity_i=8000)
    case = pm.Case(p)
    case.set_launch_shape(deposit_mode=mode)
    for s in (0, 1):
        x = _positions(np.float64 if fp64 else np.float32, np.random.default_rng(s))
        n, zero = len(x), np.zeros(len(x))
        case.set_particles(s, dict(xt=x, ux=zero, uy=zero, uz=zero, id=np.arange(n), next=np.full(n, 0xFFFFFFFF)))
    return case


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("fp64", [True, False])
@pytest.mark.parametrize("batch", [False, True])
def test_charge_just_below_a_cell_edge(pm, batch, fp64, mode):
    a, b = _case(pm, fp64, mode), _case(pm, fp64, mode)
    runs = [a, b]
    if batch:
        runs = [pm.Batch([a]), pm.Batch([b])]
        for r in runs:
            r.set_launch_shape(deposit_mode=mode, sort_interval=0)
    runs[0].step(2)
    for _ in range(2):
        runs[1].step(1)
    for case in (a, b):
        f = case.get_fields()
        for s, key in ((0, "qe"), (1, "qi")):
            assert np.array_equal(f[key], P.deposit(case.get_particles(s)["xt"], N)), (case is a, key)
    _same(a, b, "two steps")
