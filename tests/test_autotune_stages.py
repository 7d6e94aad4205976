"""The tuner times each field of a launch shape by the calls it acts on: on a model of
a device where single steps and calls of several steps have different best shapes, it
finds both (CPU only: the clock and the object are stand-ins)."""
import itertools
import json

import pytest

import workloads as W
from paper_1607_04069_amd import autotune as A


class Clock:
    now = 0.0

    def perf_counter(self):
        return self.now


class Model:
    """Steps that take longer the further a shape is from the best of their kind."""

    resident = 1024

    def __init__(self, clock, single, several, batch):
        self.clock, self.single, self.several = clock, single, several
        self.shape = dict(unroll=8, waves=0, work_groups=0, deposit_mode=1, sort_interval=25, lanes=1)
        self.steps = 0
        self.timed = []
        if batch:
            self.cases = [self]

    def launch_shape(self):
        return dict(self.shape, work_groups=self.shape["work_groups"] or self.resident)

    def set_launch_shape(self, **kw):
        self.shape = dict(self.launch_shape(), **kw)

    def sample_diagnostics(self):
        return {"particle_steps": self.steps * 1000}

    def step(self, n):
        best = self.single if n == 1 else self.several
        off = sum(self.launch_shape()[k] != v for k, v in best.items())
        self.clock.now += n * 1e-5 * (1.0 + 0.1 * off)
        self.steps += n


@pytest.fixture
def clock(monkeypatch, tmp_path):
    import torch
    monkeypatch.setattr(torch.cuda, "synchronize", lambda: None)
    monkeypatch.setattr(A, "_device", lambda: "dev")
    monkeypatch.setenv(A.CACHE_ENV, str(tmp_path / "shapes.json"))
    c = Clock()
    monkeypatch.setattr(A, "time", c)
    return c


@pytest.mark.parametrize("batch", [False, True])
@pytest.mark.parametrize("unroll,waves,part", itertools.product((8, 16), (0, 6), (1, 2)))
def test_each_field_is_timed_where_it_acts(clock, batch, unroll, waves, part):
    groups = 1024 * part if batch else 1024 // part
    single = dict(unroll=unroll, waves=waves, work_groups=groups)
    several = dict(deposit_mode=0, sort_interval=50, **(dict(lanes=3) if batch else {}))
    obj = Model(clock, single, several, batch)
    shape, rate, source = A.tune(obj, W.sweep_cases(2))
    assert source == "timed" and shape == dict(obj.launch_shape(), **single, **several)
    assert rate == pytest.approx(1000 / 1e-5)


def test_shapes_of_the_two_launch_step_are_not_looked_up(clock, tmp_path):
    obj = Model(clock, {}, {}, True)
    ps = W.sweep_cases(2)
    key = A.workload_key(obj, ps)
    old = key.replace("|" + A.STEP_FORM, "")
    assert old != key
    entry = {"shape": dict(obj.launch_shape(), work_groups=7), "particle_steps_per_s": 1.0}
    (tmp_path / "shapes.json").write_text(json.dumps({old: entry}))
    assert A.tune(obj, ps)[2] == "timed"
    assert A.tune(obj, ps)[2] == "cache"
    # the shipped shapes are of this form of the step
    assert all(f"|{A.STEP_FORM}|" in k for k in A._read(A.SHIPPED))
