"""The one-workgroup bottom of the pressure V-cycle against a plain numpy V-cycle built from the level operators, at the
edges of what it takes: segments of 1 to 4 layers and 1 to 16 of them, one-cell-wide and odd grids, a first level that is
the finest or a coarser one, one and several sweeps, and grids just past its limits (which take the per-level launches).
FP64: 1e-10 relative, as in the V-cycle test.  FP32: the error against the FP64 cycle is at most 16 times that of the
same numpy cycle carried out in FP32 (how much rounding such a cycle shows depends on the operator: its residuals cancel)."""
import numpy as np
import pytest

from test_gpu_mg import _agg, _op, _setup, _zline_ref

pytestmark = pytest.mark.gpu


def _vcycles_ref(levels, b, cycles, pre, dtype=np.float64):
    """cycles V-cycles from 0 with pre sweeps before and none after, carried out in dtype."""
    ops = [_op(d, A).astype(dtype) for d, A in levels]
    Ps = [_agg(levels[l][0], levels[l + 1][0]).astype(dtype) for l in range(len(levels) - 1)]

    def cycle(l, rhs, x):
        dims, A = levels[l]
        if l == len(levels) - 1:
            return np.linalg.solve(ops[l].toarray(), rhs)
        for _ in range(pre):
            x = _zline_ref(A, dims, x, rhs, 0)
            x = _zline_ref(A, dims, x, rhs, 1)
        return x + Ps[l] @ cycle(l + 1, Ps[l].T @ (rhs - ops[l] @ x), np.zeros(Ps[l].shape[1], dtype))

    x = np.zeros(len(b), dtype)
    for _ in range(cycles):
        x = cycle(0, b, x)
    return x


SHAPES = [(7, 5, 3),        # 2 levels, 4 segments of 1 layer, odd
          (1, 40, 5), (40, 1, 5),      # one column wide
          (12, 9, 16),      # 4 layers a segment, near the LDS limit
          (13, 10, 16),     # past it
          (3, 3, 64),       # 16 segments of 4 layers
          (3, 3, 65),       # 5 layers: not taken
          (32, 16, 2), (33, 16, 2),    # 256 columns of a colour, and more
          (16, 16, 7),      # the last segment is short
          (30, 33, 11), (61, 23, 13), (25, 60, 6)]     # the tail starts at a coarser level


@pytest.mark.parametrize("pre,cycles", [(1, 2), (3, 1), (2, 3)])
@pytest.mark.parametrize("shape", SHAPES)
def test_small_levels_match_numpy_vcycle(shape, pre, cycles):
    sim = _setup(*shape, seed=2, mg_pre=pre, mg_cycles=cycles)
    levels = sim.pressure_levels()
    b = np.random.default_rng(5).standard_normal(int(np.prod(shape)))
    x = sim.pressure_vcycle(b)
    ref = _vcycles_ref(levels, b, cycles, pre)
    err = np.max(np.abs(x - ref)) / np.max(np.abs(ref))
    assert err <= 1e-10, (shape, len(levels), err)
    # the launch has no state: the same right-hand side again gives the same result
    assert np.array_equal(sim.pressure_vcycle(b), x)


@pytest.mark.parametrize("pre,cycles", [(1, 2), (3, 1), (2, 3)])
@pytest.mark.parametrize("shape", SHAPES)
def test_small_levels_in_fp32(shape, pre, cycles):
    sim = _setup(*shape, seed=2, mg_pre=pre, mg_cycles=cycles, precision=1)
    levels = sim.pressure_levels()
    b = np.random.default_rng(5).standard_normal(int(np.prod(shape)))
    x = sim.pressure_vcycle(b)
    ref = _vcycles_ref(levels, b, cycles, pre)
    ref32 = _vcycles_ref([(d, A.astype(np.float32)) for d, A in levels], b.astype(np.float32), cycles, pre,
                         np.float32)
    err, err32 = (np.max(np.abs(v - ref)) / np.max(np.abs(ref)) for v in (x, ref32))
    assert err <= 16 * err32, (shape, len(levels), err, err32)
