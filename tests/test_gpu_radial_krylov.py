"""GPU test of Newton-Krylov solves of radial grids, whose ILU(0) factor is exact:
one Krylov iteration a Newton step, so the sweeps take no plan where one
work-group sweeps by levels, and one of short rows where a level is wider than
that; roots against the oracle within the parity tolerance of 1e-7.
"""

import numpy as np
import pytest

from oracle import polar

pytestmark = pytest.mark.gpu


def _radial(n, seed=2):
    """A random tree of n buses, loads and impedances light enough for any n."""
    import pins

    rng = np.random.default_rng(seed)
    b = np.arange(1, n)
    parents = [int(rng.integers(0, k)) for k in b]
    s = 0.2 / n
    return pins.polar_case(n, parents, list(b), [0.1 / n] * (n - 1), [0.3 / n] * (n - 1), [0.0] * (n - 1),
                           [3] + [1] * (n - 1), list(np.r_[0, -s * (0.5 + rng.random(n - 1))]),
                           list(np.r_[0, -0.4 * s * (0.5 + rng.random(n - 1))]), [1] * n)


@pytest.mark.parametrize("n,planned", [(2000, False), (2600, False), (5000, False), (15000, True)])
def test_radial(n, planned):
    from paper_1711_10579_amd import binding as B

    ctx = B.pf_ctx_create(0)
    g = _radial(n)
    ref = polar.newton(g).V
    h = B.pf_create_from(ctx, g)
    dev, _, parts = B.pf_debug_sweep_check(h, B.PF_PREC_FP64, seed=3)
    print(f"{n} buses: parts {parts}, deviation {dev:.2g}", flush=True)
    assert (min(parts) > 0) == planned and dev <= 1e-11
    for solver in (B.PF_SOLVER_GMRES, B.PF_SOLVER_BICGSTAB):
        r = B.pf_solve(h, solver=solver, max_iter=40)
        assert r.status == B.PF_CONVERGED and r.linear_iters <= 2 * r.iters
        assert np.max(np.abs(B.pf_get_voltage(h) - ref)) <= 1e-7
    h.close()
    ctx.close()


def test_mesh_without_triangles():
    """Updates of diagonal blocks only, as in a radial grid, but fill that the
    factor drops: such a mesh keeps its plan."""
    from paper_1711_10579_amd import binding as B

    import pfgen

    g = pfgen.make_polar_grid(2399, 719, 239, 11, balanced=True)
    nb = [set(map(int, g.col[g.row_ptr[i] : g.row_ptr[i + 1]])) - {i} for i in range(g.n)]
    assert not any(nb[i] & nb[j] for i in range(g.n) for j in nb[i]) and sum(map(len, nb)) > 2 * g.n
    ctx = B.pf_ctx_create(0)
    h = B.pf_create_from(ctx, g)
    dev, _, parts = B.pf_debug_sweep_check(h, B.PF_PREC_FP64, seed=3)
    print(f"parts {parts}, deviation {dev:.2g}", flush=True)
    assert min(parts) > 0 and dev <= 1e-11
    h.close()
    ctx.close()
