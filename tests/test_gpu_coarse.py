"""The dense inverse of the coarsest pressure level against numpy's, at the edges of its register tiles (multiples of 16
rows up to 96, one less and one more), on one-cell-wide grids, and just past its limit, where the general kernel takes
over.  The hierarchy is this one level, so a V-cycle is the inverse applied: 1e-10 relative in FP64, as in the V-cycle
test; in mixed precision at most 16 times the error of numpy's inverse rounded to FP32 and applied in FP32."""
import numpy as np
import pytest

from test_gpu_mg import _op, _setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [
    (2, 1, 1), (1, 1, 9), (5, 3, 1), (4, 2, 2), (1, 17, 1), (31, 1, 1), (4, 4, 2), (11, 3, 1), (1, 6, 8), (7, 7, 1),
    (4, 4, 4), (13, 5, 1), (79, 1, 1), (4, 5, 4), (9, 3, 3), (1, 1, 95), (8, 12, 1), (4, 4, 6), (97, 1, 1), (4, 6, 5)])
@pytest.mark.parametrize("precision", [0, 1])
def test_coarsest_inverse(shape, precision):
    sim = _setup(*shape, seed=4, mg_coarse=128, precision=precision)
    levels = sim.pressure_levels()
    assert len(levels) == 1
    A = _op(*levels[0]).toarray()
    b = np.random.default_rng(6).standard_normal(A.shape[0])
    ref = np.linalg.solve(A, b)
    x = sim.pressure_vcycle(b)
    scale = np.max(np.abs(ref))
    err = np.max(np.abs(x - ref)) / scale
    if precision == 0:
        assert err <= 1e-10, err
    else:
        x32 = np.linalg.inv(A).astype(np.float32) @ b.astype(np.float32)
        assert err <= 16 * max(np.max(np.abs(x32 - ref)) / scale, np.finfo(np.float32).eps), err
