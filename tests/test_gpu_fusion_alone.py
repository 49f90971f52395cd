"""A member of a fusion group computes exactly what it computes alone: its state after a step in a group equals the one
that the same simulator reaches by itself, bit for bit, on grids whose levels take each way down the V-cycle (tiles of
8 x 8, 8 x 2 and 4 x 2 columns, launches of their own, the one launch at its bottom)."""
import numpy as np
import pytest

from paper_1807_05298_amd import inputs as I
from test_gpu_fusion import _direct, _fused, _pf

pytestmark = pytest.mark.gpu

SHAPES = [(40, 40, 6), (31, 37, 23), (52, 37, 23), (60, 60, 20), (95, 96, 5), (16, 12, 20)]


@pytest.mark.parametrize("opts", [{}, {"precision": 1}, {"cpr_order": 1}, {"smoother": 0}])
def test_fused_state_is_the_direct_one(opts):
    o = _pf().default_opts(**opts)
    cases = [I.box_case(*s, seed=60, sigma=1.2, corr=(1.0, 3.0, 3.0), dts=[0.5 * I.DAY]) for s in SHAPES]
    for group in [cases] + [[c] for c in cases]:
        for c, m in zip(group, _fused(_pf(), group, o, 1)[0]):
            for name, a, b in zip("P S C Pb".split(), m, _direct(_pf(), c, o, 1)):
                assert np.array_equal(a, b), (c.name, len(group), name)


@pytest.mark.parametrize("opts", [{}, {"precision": 1}, {"smoother": 0}])
def test_members_that_share_the_cache(opts):
    """Six members of 101k cells: together their copies of J are too large for the memory-side cache, one's is not."""
    pf = _pf()
    o = pf.default_opts(**opts)
    c = I.box_case(58, 58, 30, seed=61, dts=[0.5 * I.DAY])
    ref = _direct(pf, c, o, 1)
    for m in _fused(pf, [c] * 6, o, 1)[0]:
        assert all(np.array_equal(a, b) for a, b in zip(m, ref))
