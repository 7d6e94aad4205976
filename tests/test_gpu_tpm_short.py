"""Flights of few events, or of steps that mostly collide, take fewer lanes an atom and
longer runs of atoms (runs on an MI355X): on both sides of each limit an atom's flight
is that of a launch with one lane per atom."""
import numpy as np
import pytest

from test_gpu_tpm_lanes import N_ONE_LANE, _inputs, pm  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("e_max", [1, 8, 15, 16, 64, 127, 512])
def test_event_limits_do_not_change_an_atom(pm, e_max, mode):
    kw = dict(p_pa=5.0, mode=mode, dt_s=1e-7, e_max=e_max, scatter=mode)
    big = pm.run_test_particles(*_inputs(N_ONE_LANE, **kw), trace=True)["trace"]
    for n, first in ((1, 5), (63, 100), (4097, 1000), (66_000, 30_001)):
        small = pm.run_test_particles(*_inputs(n, first, **kw), trace=True)
        for k, v in small["trace"].items():
            assert np.array_equal(v, big[k][first:first + n], equal_nan=v.dtype.kind == "f"), (n, k)
        assert small["events"] == int(small["trace"]["events"].astype(np.int64).sum())
        assert small["n_unfinished"] == int((small["trace"]["wall"] == 2).sum())


# less than one event an atom; less than 16; a fixed step's probability at the majorant
# (per step of 1 us at 1 Pa: 0.32) that leaves 32, 8, 4 and 2 lanes
@pytest.mark.parametrize("kw", [dict(p_pa=0.0), dict(p_pa=0.15), dict(p_pa=0.25), dict(p_pa=0.9), dict(p_pa=1.1),
                                dict(p_pa=1.0, dt_s=1e-6), dict(p_pa=5.0, dt_s=1e-6), dict(p_pa=5.0, dt_s=3e-6),
                                dict(p_pa=5.0, dt_s=1e-4)])
def test_short_and_dense_flights_do_not_change_an_atom(pm, kw):
    big = pm.run_test_particles(*_inputs(N_ONE_LANE, **kw), trace=True)["trace"]
    for n, first in ((1, 5), (63, 100), (4097, 1000), (66_000, 30_001), (262_145, 200_000)):
        small = pm.run_test_particles(*_inputs(n, first, **kw), trace=True)
        for k, v in small["trace"].items():
            assert np.array_equal(v, big[k][first:first + n], equal_nan=v.dtype.kind == "f"), (n, k)
        assert small["n_target"] == int((small["trace"]["wall"] == 0).sum())


# the box and low event limits with few and with many collisions an event: one lane, 16 and between
@pytest.mark.parametrize("omega", [0.55, 0.99])
@pytest.mark.parametrize("kw", [dict(mode=1, e_max=150), dict(mode=1, e_max=40), dict(mode=0, e_max=150),
                                dict(mode=1, e_max=300, dt_s=1e-6)])
def test_boxes_and_limits_do_not_change_an_atom(pm, kw, omega):
    def flight(n, first=0):
        src, tp = _inputs(n, first, p_pa=3.0, **kw)
        return pm.run_test_particles(src, dict(tp, omega=omega), trace=True)
    big = flight(N_ONE_LANE)["trace"]
    for n, first in ((1, 5), (63, 100), (4097, 1000), (16_500, 3), (33_000, 70_000), (66_000, 30_001)):
        small = flight(n, first)
        for k, v in small["trace"].items():
            assert np.array_equal(v, big[k][first:first + n], equal_nan=v.dtype.kind == "f"), (n, k)
        assert small["events"] == int(small["trace"]["events"].astype(np.int64).sum())
