"""The launch that takes a V-cycle down one level gives, bit for bit, the values of the three launches it replaces (a
segment length set by the caller, here the same two layers, keeps those), so that the route never shows in a result: from
x = 0 and from another cycle's x, one and two sweeps, both precisions, whole and ragged tiles, low and tall levels.  A
large coarsest level keeps the bottom of the cycle the same in both."""
import numpy as np
import pytest

from test_gpu_mg import _pf, _setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("pre,cycles", [(1, 1), (1, 3), (2, 2)])
@pytest.mark.parametrize("shape", [(97, 190, 5), (49, 95, 5), (57, 47, 1), (41, 33, 2), (24, 23, 5), (52, 37, 23),
                                   (31, 60, 39), (101, 37, 36)])
def test_down_launch_is_bitwise_the_three(shape, pre, cycles, precision):
    pf = _pf()
    b = np.random.default_rng(10).standard_normal(int(np.prod(shape)))
    x = []
    for zline_len in (0, 2):
        sim = _setup(*shape, seed=4, mg_pre=pre, mg_cycles=cycles, mg_coarse=1000, precision=precision,
                     zline_len=zline_len)
        down = [c for c in range(cycles) for r in sim.pressure_route(c) if r[0] == pf.MG_DOWN]
        assert zline_len == 0 or not down
        assert zline_len or down or (pre == 2 and shape[2] > 30)     # (tall levels with two sweeps keep the three)
        x.append(sim.pressure_vcycle(b))
    assert np.array_equal(x[0], x[1])
