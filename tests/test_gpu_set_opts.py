"""pf_set_opts and the workspace's plan: a simulator created with block Jacobi has no room for red-black ILU(0)'s
factors, so that smoother is refused and the simulator goes on as it was; the other way round is accepted, there and
back."""
import numpy as np
import pytest

from paper_1807_05298_amd import inputs as I
from test_gpu_fusion import _pf

pytestmark = pytest.mark.gpu

CASE = I.box_case(13, 9, 4, seed=5, dts=[0.5 * I.DAY])


def _stepped(sim):
    sim.set_state(CASE.P0, CASE.S0, CASE.C0, CASE.Pb0)
    sim.step(float(CASE.dts[0]))
    return sim.get_state()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("order", [0, 1])
def test_smoother_may_not_outgrow_the_workspace(precision, order):
    pf = _pf()
    bjac = pf.default_opts(precision=precision, cpr_order=order, smoother=pf.SMOOTH_BJAC)
    ilu = pf.default_opts(precision=precision, cpr_order=order, smoother=pf.SMOOTH_RBILU0)
    a, b = pf.Simulator(CASE, bjac), pf.Simulator(CASE, ilu)
    want, want_ilu = _stepped(a), _stepped(b)
    with pytest.raises(pf.PFError) as e:
        a.set_opts(ilu)
    assert e.value.status == pf.PF_EINVAL
    assert all(np.array_equal(x, y) for x, y in zip(_stepped(a), want))
    b.set_opts(bjac)
    assert all(np.array_equal(x, y) for x, y in zip(_stepped(b), want))
    b.set_opts(ilu)
    assert all(np.array_equal(x, y) for x, y in zip(_stepped(b), want_ilu))
