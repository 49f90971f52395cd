"""The launch that takes a V-cycle down one level (colour-1 half-sweep, residual restriction, the next level's first
colour-0 half-sweep) against a plain numpy V-cycle built from the level operators, at the edges of what it takes: whole
and ragged grids of each of its tiles, one layer, as many as it takes and more (separate launches); one sweep from zero (lateral residuals) and several cycles or sweeps (full
residuals).  FP64: 1e-10 relative, as in the V-cycle test; FP32: at most 16 times the error of the numpy cycle in FP32."""
import numpy as np
import pytest

from test_gpu_mg import _setup
from test_gpu_mg_tail import _vcycles_ref

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("pre,cycles", [(1, 2), (2, 2)])
@pytest.mark.parametrize("shape", [
    (97, 190, 5), (96, 192, 5),                                   # tiles of 8 x 8 columns
    (49, 95, 5), (100, 44, 6), (57, 47, 1),                       # of 8 x 2
    (40, 32, 2), (41, 33, 2), (24, 23, 5), (64, 16, 12), (5, 60, 20), (16, 17, 20), (8, 8, 30),      # of 4 x 2
    (9, 7, 40), (33, 26, 47)])                                    # launches of their own on the first level
def test_down_launch_matches_numpy_vcycle(shape, pre, cycles, precision):
    sim = _setup(*shape, seed=3, mg_pre=pre, mg_cycles=cycles, precision=precision)
    levels = sim.pressure_levels()
    assert len(levels) > 1
    b = np.random.default_rng(9).standard_normal(int(np.prod(shape)))
    x = sim.pressure_vcycle(b)
    ref = _vcycles_ref(levels, b, cycles, pre)
    err = np.max(np.abs(x - ref)) / np.max(np.abs(ref))
    if precision == 0:
        assert err <= 1e-10, (shape, len(levels), err)
    else:
        ref32 = _vcycles_ref([(d, A.astype(np.float32)) for d, A in levels], b.astype(np.float32), cycles, pre,
                             np.float32)
        err32 = np.max(np.abs(ref32 - ref)) / np.max(np.abs(ref))
        assert err <= 16 * err32, (shape, len(levels), err, err32)
    # the launch has no state
    assert np.array_equal(sim.pressure_vcycle(b), x)
