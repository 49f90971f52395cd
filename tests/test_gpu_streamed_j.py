"""The kernels that stream J load it past the caches by its size, a fusion group's all together.  A simulator too small
for that by itself takes the plain variants alone, which the other tests check on such grids, and the streamed ones in a
group of eight: its linear solve has to be the same bit for bit, on grids with pad slots (odd nx), one cell in x, one row
and one layer, for every path that has the two variants; restarts take the natural-order product too."""
import threading

import numpy as np
import pytest

from paper_1807_05298_amd import inputs as I
from test_gpu_fusion import _pf
from test_gpu_precond import _setup

pytestmark = pytest.mark.gpu


def _each(calls):
    """One thread a call: a member of a group waits for the others to come to a point where they wait too."""
    out = [None] * len(calls)

    def run(k):
        out[k] = calls[k]()

    th = [threading.Thread(target=run, args=(k,)) for k in range(len(calls))]
    for t in th:
        t.start()
    for t in th:
        t.join()
    return out


def _join(pf, fu, sims):
    for s in sims:
        assert pf._lib.pf_fusion_join(fu.h, s.h) == pf.PF_OK


@pytest.mark.parametrize("opts", [{"restart": 2}, {"precision": 1}, {"cpr_order": 1}, {"smoother": 0}])
@pytest.mark.parametrize("shape", [(43, 47, 41), (1, 300, 280), (301, 1, 281), (301, 281, 1)])
def test_streamed_variants_are_bitwise_the_plain_ones(shape, opts):
    pf = _pf()
    sims = [_setup(shape, 31, **opts)[0] for _ in range(8)]
    b = np.random.default_rng(32).standard_normal(sims[0].nv)
    assert sims[0].streams_j() == (False, False)
    want, its, rel = sims[0].linear_solve(b, 1e-9)
    fu = pf.Fusion()
    _join(pf, fu, sims)
    assert sims[0].streams_j() == (True, True)
    got = _each([lambda s=s: s.linear_solve(b, 1e-9) for s in sims])
    _each([lambda s=s: pf._lib.pf_fusion_leave(s.h) for s in sims])
    assert its == 5
    for x, i, r in got:
        assert np.array_equal(x, want) and i == its and r == rel
    fu.close()


def test_line_counts_a_group_together():
    pf = _pf()
    c = I.box_case(58, 58, 30, seed=61)         # 33.9 MB of colour-split copies, 45.2 MB of natural-order planes
    sims = [pf.Simulator(c, pf.default_opts()) for _ in range(6)]
    fu = pf.Fusion()
    got = []
    for s in sims:
        got.append(sims[0].streams_j())
        _join(pf, fu, [s])
    assert got == [(False, False)] * 5 + [(True, True)]
    _each([lambda s=s: pf._lib.pf_fusion_leave(s.h) for s in sims])
    assert sims[0].streams_j() == (False, False)
    fu.close()
