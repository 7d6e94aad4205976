"""A population far above the one its case was loaded with (runs on an MI355X): the
one-launch steps take their workgroups from the capacity then, and give what single
steps give, bit for bit."""
import numpy as np
import pytest

import workloads as W
from test_gpu_fused import _same, pm  # noqa: F401  (the fixture)

pytestmark = pytest.mark.gpu


def _grown(pm, fp64, np_each, capacity):
    big = W.discharge(0.025, 64, 100.0, 400, 5.0, 9001, 1e15, seed=4, case_id=2, fp64=fp64)
    one = pm.Case(big)
    st = [one.get_particles(s) for s in (0, 1)]
    one.close()
    out = []
    for _ in range(2):
        out.append(pm.Case(dict(big, np_e=np_each, np_i=np_each, n0_m3=1e15 * np_each / 9001, capacity_e=capacity,
                                capacity_i=capacity)))
        for s in (0, 1):
            out[-1].set_particles(s, st[s])
    return out


# workgroups by the load, by the capacity with fewer of them than passes, and more
@pytest.mark.parametrize("fp64", [True, False])
@pytest.mark.parametrize("np_each,capacity", [(100, 12_000), (1, 40_000), (100, 3_000_000)])
def test_outgrown_load(pm, np_each, capacity, fp64):
    a, b = _grown(pm, fp64, np_each, capacity)
    c, d = _grown(pm, fp64, np_each, capacity)
    fused, plain = pm.Batch([c]), pm.Batch([d])
    for n in (2, 1, 26):
        for x, y in ((a, b), (fused, plain)):
            x.step(n)
            for _ in range(n):
                y.step(1)
        _same(a, b, n)
        _same(c, d, ("batch", n))
