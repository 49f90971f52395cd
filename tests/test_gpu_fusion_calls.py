"""Every call that returns host data, made by a member of a fusion group on a thread of its own: the data are those of the
work recorded before the call, as alone, bit for bit.  (The calls of one member are not those of another at the same
time: the second starts with another state.)"""
import threading

import numpy as np
import pytest

from paper_1807_05298_amd import inputs as I
from test_gpu_fusion import _pf

pytestmark = pytest.mark.gpu


def _calls(pf, sim, seed):
    """What a program that drives its own loop gets back, in order."""
    rng = np.random.default_rng(seed)
    c, out = sim.case, []
    b = rng.standard_normal(sim.nv)
    if seed % 2:
        sim.set_equilibrium_state(c.top + 3.0, 210e5, c.top + 10.0)
        out += list(sim.get_state())
    sim.set_state(c.P0, c.S0, c.C0, c.Pb0)
    sim.begin_step()
    out += list(sim.assemble(float(c.dts[0])))
    x, its, rel = sim.linear_solve(b, 1e-6)
    out += [x, np.array([its, rel]), sim.spmv(x), *sim.precond_apply(b), sim.smoother_apply(b),
            sim.pressure_vcycle(b[:sim.n])]
    out += [A for _, A in sim.pressure_levels()] + [sim.static()[k] for k in ("row_scale", "Tx", "PVr", "perf_wi")]
    sim.step(float(c.dts[0]))
    out += list(sim.get_state())
    w = sim.well_status()
    return out + [np.asarray(w[k]) for k in sorted(w)]


@pytest.mark.parametrize("opts", [{}, {"precision": 1}, {"cpr_order": 1, "smoother": 0}])
def test_results_of_calls_in_a_group(opts):
    pf = _pf()
    o = pf.default_opts(**opts)
    cases = [I.box_case(13, 9, 4, seed=6, dts=[0.5 * I.DAY]), I.box_case(24, 20, 5, seed=7, dts=[0.5 * I.DAY])]
    want = []
    for k, c in enumerate(cases):
        sim = pf.Simulator(c, o)
        want.append(_calls(pf, sim, k))
        sim.close()
    sims = [pf.Simulator(c, o) for c in cases]
    fu, got, err = pf.Fusion(), [None, None], []
    for s in sims:
        assert pf._lib.pf_fusion_join(fu.h, s.h) == pf.PF_OK

    def run(k):
        try:
            got[k] = _calls(pf, sims[k], k)
        except Exception as e:          # the other member must not be left waiting
            err.append(e)
        pf._lib.pf_fusion_leave(sims[k].h)

    th = [threading.Thread(target=run, args=(k,)) for k in range(2)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    assert not err, err
    for k in range(2):
        assert len(got[k]) == len(want[k])
        for q, (a, b) in enumerate(zip(got[k], want[k])):
            assert np.array_equal(a, b), (k, q)
    for s in sims:
        s.close()
    fu.close()
