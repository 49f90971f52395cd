"""zline_len, the layers of a smoother segment, holds on every level: a caller who sets it gets the launches that take
it, not the merged ones whose segments are their own, and the same V-cycle (numpy, 1e-10 as in the V-cycle test)."""
import numpy as np
import pytest

from test_gpu_mg import _pf, _setup
from test_gpu_mg_tail import _vcycles_ref

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("zline_len", [1, 2, 4, 8, 30])
@pytest.mark.parametrize("shape", [(10, 8, 3), (31, 37, 23), (97, 90, 5), (9, 7, 40)])
def test_segment_length_holds_on_every_level(shape, zline_len):
    pf = _pf()
    merged = {pf.MG_DOWN, pf.MG_TAIL}
    assert merged & {r[0] for r in _setup(*shape, mg_pre=1).pressure_route()}
    sim = _setup(*shape, mg_pre=1, mg_cycles=2, zline_len=zline_len)
    for cycle in (0, 1):
        assert not merged & {r[0] for r in sim.pressure_route(cycle)}
    b = np.random.default_rng(4).standard_normal(int(np.prod(shape)))
    ref = _vcycles_ref(sim.pressure_levels(), b, 2, 1)
    assert np.max(np.abs(sim.pressure_vcycle(b) - ref)) <= 1e-10 * np.max(np.abs(ref))
