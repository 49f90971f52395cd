"""Where the launch that takes a V-cycle down one level runs, and that it is right there: the route of every level of
columns of up to 39 layers (20 segments of a line, 10 of the next level's) for each of its tiles that takes them, and of
the first grid past its limit, against the numpy V-cycle with the bounds of the test on low levels."""
import numpy as np
import pytest

from test_gpu_mg import _pf, _setup
from test_gpu_mg_tail import _vcycles_ref

pytestmark = pytest.mark.gpu

# tile and, with +, the next level's half-sweep; s: launches of their own; T: the bottom in one
CASES = [((97, 190, 5), 0, ["8x8+", "8x2+", "4x2", "T", "T", "T"]),
         ((31, 37, 23), 0, ["4x2+", "4x2", "T", "T"]),
         ((52, 37, 23), 1, ["4x2+", "4x2", "T", "T", "T"]),
         ((31, 60, 39), 0, ["4x2+", "s", "T", "T", "T"]),
         ((31, 60, 40), 0, ["s", "s", "T", "T", "T"]),
         ((101, 37, 36), 0, ["8x2+", "4x2+", "4x2", "T", "T"]),
         ((101, 37, 38), 0, ["s", "4x2+", "4x2", "T", "T"]),
         ((101, 37, 38), 1, ["8x2+", "4x2+", "4x2", "T", "T"]),
         ((101, 77, 33), 0, ["s", "4x2+", "4x2+", "4x2", "T", "T"])]


@pytest.mark.parametrize("shape,precision,want", CASES)
def test_route_and_vcycle(shape, precision, want):
    pf = _pf()
    sim = _setup(*shape, seed=3, mg_pre=1, mg_cycles=2, precision=precision)
    name = {pf.MG_SWEEPS: "s", pf.MG_WHOLE: "w", pf.MG_TAIL: "T", pf.MG_DENSE: "d"}
    assert [name.get(k) or f"{tx}x{ty}" + "+" * nxt for k, tx, ty, nxt in sim.pressure_route()] == want
    levels = sim.pressure_levels()
    b = np.random.default_rng(9).standard_normal(int(np.prod(shape)))
    x = sim.pressure_vcycle(b)
    ref = _vcycles_ref(levels, b, 2, 1)
    err = np.max(np.abs(x - ref)) / np.max(np.abs(ref))
    if precision == 0:
        assert err <= 1e-10, err
    else:
        ref32 = _vcycles_ref([(d, A.astype(np.float32)) for d, A in levels], b.astype(np.float32), 2, 1, np.float32)
        assert err <= 16 * np.max(np.abs(ref32 - ref)) / np.max(np.abs(ref)), err
