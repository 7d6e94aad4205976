"""Batches on both sides of the size up to which several steps of a call are fused, and
with fewer workgroups than their members' shares (runs on an MI355X): every member is
what it is alone."""
import numpy as np
import pytest

import workloads as W
from test_gpu_fused import pm  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


def _params(np_each, k):
    return W.discharge(0.04, 128, 200.0, 400, 0.5, np_each, 4e15, seed=11, case_id=k, fp64=True, capacity_factor=1.1,
                       sort_interval=10)


def _same(a, b, label):
    for read in ("get_fields", "sample_diagnostics"):
        u, v = getattr(a, read)(), getattr(b, read)()
        for k in u:
            assert np.array_equal(u[k], v[k], equal_nan=True), (label, read, k)


def test_slotted_batch_across_the_size(pm):
    """10.4M FP64 particles (above 40k for each of 256 resident workgroups), then half of
    them, then all again, through captured cycles and plain steps."""
    sizes = (2_600_000, 2_600_000, 3000)
    alone = [pm.Case(_params(n, k)) for k, n in enumerate(sizes)]
    members = [pm.Case(_params(n, k)) for k, n in enumerate(sizes)]
    b = pm.SlotBatch(8, 400, fp64=True)
    b.set_launch_shape(lanes=1, sort_interval=10)
    for k, m in enumerate(members):
        b.set_slot(2 * k, m)
    present = {0, 1, 2}
    for turn, leaves in enumerate((None, 1, None)):
        print(f"turn {turn}", flush=True)
        if leaves is not None:
            b.set_slot(2 * leaves, None)
            present.remove(leaves)
        elif turn:
            b.set_slot(2, members[1])
            present.add(1)
        b.step_rf_cycles(1)
        b.step(13)
        for k in present:
            alone[k].step(413)
        for k, (u, v) in enumerate(zip(alone, members)):
            _same(u, v, (turn, k))
    b.close()


@pytest.mark.parametrize("m,lanes", [(300, 1), (1000, 3)])
def test_more_members_than_workgroups_of_a_share(pm, m, lanes):
    """As many members as leave each one or two workgroups, and more than there are."""
    sizes = [int(s) for s in np.random.default_rng(m).integers(1, 6000, m)]
    cases = [pm.Case(_params(n, k)) for k, n in enumerate(sizes)]
    b = pm.Batch(cases)
    b.set_launch_shape(lanes=lanes, sort_interval=10)
    b.step(12)
    for k in (0, 1, m // 2, m - 1, int(np.argmax(sizes)), int(np.argmin(sizes))):
        one = pm.Case(_params(sizes[k], k))
        one.step(12)
        _same(one, cases[k], k)
    b.close()
