"""Launch shapes where they act (runs on an MI355X): the push variants in single steps
and in time_kernels, the workgroup limit in single steps and in calls of several.  The
state is that of the default shape, whatever the shape."""
import time

import pytest

import workloads as W
from test_gpu_fused import _same, pm  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu

SHAPES = [dict(unroll=16), dict(waves=6), dict(unroll=16, waves=6, deposit_mode=0), dict(work_groups=3),
          dict(sort_interval=7, unroll=16, waves=6, work_groups=1), dict(lanes=2, unroll=16),
          dict(lanes=3, waves=6, work_groups=5)]


def _cases(pm, fp64):
    return [pm.Case(W.discharge(0.025, n_cells, 100.0 + k, 200, 3.0, np_each, 1e15, seed=7, case_id=k, fp64=fp64))
            for k, (np_each, n_cells) in enumerate(((20_011, 64), (3000, 777), (1, 1), (9000, 1024)))]


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("k", range(len(SHAPES)))
def test_shapes_of_single_steps(pm, k, fp64):
    a, b = _cases(pm, fp64), _cases(pm, fp64)
    for x, y in zip(a, b):
        y.set_launch_shape(**{key: v for key, v in SHAPES[k].items() if key != "lanes"})
        x.step(10)
        for _ in range(8):
            y.step(1)
        y.time_kernels(2)
        _same(x, y, SHAPES[k])
    a, b = _cases(pm, fp64), _cases(pm, fp64)
    plain, shaped = pm.Batch(a), pm.Batch(b)
    shaped.set_launch_shape(**SHAPES[k])
    plain.step(10)
    for _ in range(8):
        shaped.step(1)
    shaped.time_kernels(2)
    for x, y in zip(a, b):
        _same(x, y, ("batch", SHAPES[k]))


def test_one_working_workgroup_in_single_steps(pm):
    """200k particles for one working workgroup: those that only hold slots take what
    is beyond its 65532."""
    p = W.discharge_working(np_each=100_000)
    a, b = pm.Case(p), pm.Case(p)
    b.set_launch_shape(work_groups=1, sort_interval=7)
    a.step(15)
    for _ in range(15):
        b.step(1)
    _same(a, b, "one workgroup")


def _time(torch, f):
    f()
    best = 1e9
    for _ in range(3):
        torch.cuda.synchronize()
        t = time.perf_counter()
        f()
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    return best


@pytest.mark.parametrize("kind", ["case", "batch", "slots"])
def test_several_steps_keep_the_workgroup_limit(pm, kind):
    """Two workgroups take about fifty passes each where one per pass is a hundred of
    them: several times as long, and the same state."""
    import torch
    p = W.discharge_working(np_each=100_000)
    a, b = pm.Case(p), pm.Case(p)
    free, held = a, b
    if kind == "batch":
        free, held = pm.Batch([a]), pm.Batch([b])
    elif kind == "slots":
        free, held = (pm.SlotBatch(2, p["steps_per_cycle"]) for _ in range(2))
        free.set_slot(0, a)
        held.set_slot(0, b)
    for x, n in ((free, 0), (held, 2)):
        x.set_launch_shape(work_groups=n, sort_interval=25)
    t_free, t_held = (_time(torch, lambda: x.step(25)) for x in (free, held))
    _same(a, b, kind)
    assert t_held > 3 * t_free, (t_held, t_free)
    held.set_launch_shape(work_groups=0)
    assert _time(torch, lambda: held.step(25)) < t_held / 3


@pytest.mark.parametrize("fp64", [False, True])
def test_default_workgroups_of_a_large_case(pm, fp64):
    """At most five on a CU (three in FP64), whatever the registers allow: more of them
    stream slower."""
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    c = pm.Case(W.discharge_working(fp64=fp64))
    for sh in (dict(), dict(unroll=8, waves=6), dict(unroll=16, waves=0)):
        c.set_launch_shape(work_groups=0, **sh)
        assert 256 < c.launch_shape()["work_groups"] <= (3 if fp64 else 5) * cus
