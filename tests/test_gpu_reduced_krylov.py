"""FGMRES with Krylov vectors of the black cells and wells alone (FP64, red-black ILU(0), pressure first; the red part of
every vector is a multiple of the cycle's residual's) against a plain numpy FGMRES on whole vectors, which takes
z = M^{-1} v from pf_precond_apply and J z from pf_spmv.  Both minimise the residual over the same space, so the two
residuals differ by rounding alone: |J (x - x_ref)| <= 1e-9 |b|, a few thousand roundings of the column operations
amplified by the condition of the preconditioned operator.  Right-hand sides that are wholly red, wholly black or wells
alone, one-cell-wide and odd grids, restarts, the second Gram-Schmidt pass, post-smoothing, one and three V-cycles, a
pressure hierarchy that is one launch and one that is not."""
import numpy as np
import pytest

from test_gpu_precond import _setup

pytestmark = pytest.mark.gpu


def _fgmres(sim, b, its, restart):
    """its iterations from 0 (modified Gram-Schmidt, twice)."""
    x = np.zeros_like(b)
    while its > 0:
        r = b - sim.spmv(x)
        m = min(restart, its)
        V, Z = [r / np.linalg.norm(r)], []
        H = np.zeros((m + 1, m))
        for j in range(m):
            Z.append(sim.precond_apply(V[j])[0])
            w = sim.spmv(Z[j])
            for _ in range(2):
                for k in range(j + 1):
                    h = V[k] @ w
                    H[k, j] += h
                    w = w - h * V[k]
            H[j + 1, j] = np.linalg.norm(w)
            V.append(w / H[j + 1, j])
        g = np.zeros(m + 1)
        g[0] = np.linalg.norm(r)
        y = np.linalg.lstsq(H, g, rcond=None)[0]
        x = x + np.array(Z).T @ y
        its -= m
    return x


@pytest.mark.parametrize("part", ["all", "red", "black", "wells"])
@pytest.mark.parametrize("shape,opts", [
    ((10, 8, 3), {}), ((7, 5, 11), {"restart": 3}), ((1, 12, 20), {"reorth": 1}), ((15, 1, 9), {"mg_cycles": 3}),
    ((21, 9, 1), {"restart": 2, "reorth": 1}), ((31, 26, 6), {}), ((31, 26, 6), {"mg_post": 1, "mg_cycles": 1}),
    ((13, 9, 4), {"mg_post": 2, "restart": 4}), ((40, 33, 9), {"mg_cycles": 1, "restart": 4}), ((3, 3, 70), {})])
def test_black_cell_vectors_match_whole_ones(shape, opts, part):
    sim, _ = _setup(shape, 7, **opts)
    n, case = sim.n, sim.case_
    b = np.random.default_rng(8).standard_normal(sim.nv)
    iz, rem = np.divmod(np.arange(n), case.nx * case.ny)
    iy, ix = np.divmod(rem, case.nx)
    red = np.tile((ix + iy + iz) % 2 == 0, 3)
    keep = {"all": np.ones(sim.nv, bool), "red": np.append(red, np.zeros(sim.nv - 3 * n, bool)),
            "black": np.append(~red, np.zeros(sim.nv - 3 * n, bool)), "wells": np.arange(sim.nv) >= 3 * n}[part]
    b[~keep] = 0.0
    x, its, rel = sim.linear_solve(b, 1e-6)      # 5 iterations at most
    ref = _fgmres(sim, b, its, opts.get("restart", 30))
    nb = np.linalg.norm(b)
    assert its >= 1 and np.linalg.norm(sim.spmv(x - ref)) <= 1e-9 * nb
    assert abs(np.linalg.norm(b - sim.spmv(x)) / nb - rel) <= 1e-9
    x2, its2, rel2 = sim.linear_solve(b, 1e-6)
    assert its2 == its and rel2 == rel and np.array_equal(x2, x)
