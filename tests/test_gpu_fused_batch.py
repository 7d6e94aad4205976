"""Several steps of a batch in one call run in one launch each, a single step in two
(runs on an MI355X): both give the same particles, charge, field and diagnostics,
bit for bit, whatever the lanes, slots and members."""
import numpy as np
import pytest

import workloads as W
from test_gpu_fused import _same, pm  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu

SIZES = [(5000, 64, 1.0), (1, 1, 5.0), (2047, 777, 10.0), (40_000, 1024, 0.5), (2049, 129, 300.0), (300, 33, 20.0)]


def _members(pm, n, fp64):
    out = []
    for k in range(n):
        np_each, cells, p_pa = SIZES[k % len(SIZES)]
        out.append(pm.Case(W.discharge(0.025, cells, 100.0 + k, 200, p_pa, np_each, 1e15, seed=3, case_id=k, fp64=fp64,
                                       capacity_factor=8)))
    return out


def _all_same(a, b, label):
    for k, (u, v) in enumerate(zip(a, b)):
        _same(u, v, (label, k))


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("n,lanes,sort", [(1, 1, 7), (6, 1, 25), (6, 3, 0), (13, 4, 3)])
def test_batch(pm, n, lanes, sort, fp64):
    a, b = _members(pm, n, fp64), _members(pm, n, fp64)
    fused, plain = pm.Batch(a), pm.Batch(b)
    for x in (fused, plain):
        x.set_launch_shape(lanes=lanes, sort_interval=sort)
    for k in (1, 2, 3, 26):
        print(f"{n} members, {lanes} lanes: {k} steps", flush=True)
        fused.step(k)
        for _ in range(k):
            plain.step(1)
        _all_same(a, b, k)
    fused.close()
    plain.close()


@pytest.mark.parametrize("slots,lanes", [(8, 2), (700, 3)])
def test_slots_and_cycles(pm, slots, lanes):
    """Members that come and go between captured cycles, and more slots than
    workgroups fit on the device."""
    a, b = _members(pm, 6, False), _members(pm, 6, False)
    fused, plain = pm.SlotBatch(slots, 200), pm.SlotBatch(slots, 200)
    for x in (fused, plain):
        x.set_launch_shape(lanes=lanes, sort_interval=50)
    places = [0, 1, 2, 3, slots - 2, slots - 1]
    for k in range(4):
        fused.set_slot(places[k], a[k])
        plain.set_slot(places[k], b[k])
    for turn in range(3):
        print(f"{slots} slots, cycle {turn}", flush=True)
        fused.step_rf_cycles(1)
        for _ in range(200):
            plain.step(1)
        _all_same(a, b, turn)
        for s, m in ((places[turn], None), (places[turn + 3], turn + 3)):
            fused.set_slot(s, None if m is None else a[m])
            plain.set_slot(s, None if m is None else b[m])
    fused.close()
    plain.close()
