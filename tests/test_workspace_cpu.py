"""pf_workspace_size on the host: what red-black ILU(0) takes over block Jacobi in FP64 is its factors, its copies of J and
the well border's map in their layout (each array is aligned to 256 bytes), and nothing of it is in a block-Jacobi plan."""
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.skipif(
    not os.path.exists(os.path.join(ROOT, "paper_1807_05298_amd", "libpolyflood.so")), reason="library not built")


@pytest.mark.parametrize("shape", [(40, 32, 20), (41, 33, 21), (1, 200, 90)])
def test_smoother_share_of_the_workspace(shape):
    from paper_1807_05298_amd import inputs as I
    from paper_1807_05298_amd import polyflood as pf
    case = I.box_case(*shape)
    n, ns = case.n, (shape[0] + 1) // 2 * shape[1] * shape[2]
    size = [pf.workspace_size(case, pf.default_opts(smoother=s)) for s in (pf.SMOOTH_BJAC, pf.SMOOTH_RBILU0)]
    factors = 8 * (18 * ns - 9 * n)
    copies = 8 * (2 * ((ns + 63) // 64 * 64 * 6 * 7) + 18 * ns)
    border_map = 4 * 2 * ns
    assert abs(size[1] - size[0] - (factors + copies + border_map)) <= 4 * 256
