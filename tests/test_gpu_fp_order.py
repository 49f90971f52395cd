"""Algorithm 2's stage order in FP64, with the residual between the stages (v - J y with the well border) from one
launch.  z against the hooks composed on the host,
  y = S^{-1} v,  t = v - J y,  p = V-cycles(Pi_r t),  pb = (t_w - sum C p) / D_w,  z = y + (p, 0, 0; pb),
to 1e-9, as for the other order, and w against pf_spmv(z) to 1e-12 of its largest entry; one-cell-wide and odd grids,
cells not a multiple of a block, both smoothers, several perforations a well."""
import numpy as np
import pytest

from test_gpu_precond import _setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("smoother", [0, 1])
@pytest.mark.parametrize("shape", [(13, 9, 4), (1, 12, 20), (15, 1, 9), (21, 9, 1), (16, 8, 2), (31, 26, 6)])
def test_stages_and_product(shape, smoother):
    sim, border = _setup(shape, 21, cpr_order=1, smoother=smoother)
    n, nw = sim.n, sim.nw
    v = np.random.default_rng(22).standard_normal(sim.nv)
    z, w = sim.precond_apply(v)
    ref_w = sim.spmv(z)
    assert np.max(np.abs(w - ref_w)) <= 1e-12 * np.max(np.abs(ref_w))
    st = sim.static()
    y = sim.smoother_apply(v)
    t = v - sim.spmv(y)
    p = sim.pressure_vcycle(t[:n] + t[n:2 * n])
    Dw, s = np.zeros(nw), np.zeros(nw)
    Dw[st["perf_well"]] = border[:, 6]
    np.add.at(s, st["perf_well"], border[:, 3] * p[st["perf_cell"]])
    ref = y.copy()
    ref[:n] += p
    ref[3 * n:] += (t[3 * n:] - s) / Dw
    assert np.max(np.abs(z - ref)) <= 1e-9 * np.max(np.abs(ref))
    z2, w2 = sim.precond_apply(v)
    assert np.array_equal(z, z2) and np.array_equal(w, w2)
