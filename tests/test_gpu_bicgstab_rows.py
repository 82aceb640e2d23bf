"""GPU test of BiCGStab's matrix products with a lane a row, the form of batches
with room for many more rows than their grids have (past 204,800): a large grid
beside many small ones, with rows of one to forty blocks (a star's middle) and
instances of one row to a whole chunk of 256 and one more.  The grids alone take
four lanes a row; every result is bit-identical to its solve alone.
"""

import numpy as np
import pytest

import pfgen

pytestmark = pytest.mark.gpu


def _mesh(n):
    return pfgen.make_polar_grid(n, (3 * n) // 10, n // 10, 11, balanced=True)


def _star(n):
    import pins

    b = np.arange(1, n)
    s = 0.2 / n
    return pins.polar_case(n, [1] * (n - 2) + [0], list(b[1:]) + [1], [0.1 / n] * (n - 1), [0.3 / n] * (n - 1),
                           [0.0] * (n - 1), [3] + [1] * (n - 1), [0.0] + [-s] * (n - 1), [0.0] + [-0.4 * s] * (n - 1),
                           [1] * n)


@pytest.mark.parametrize("mixed", [False, True], ids=["fp64", "mixed"])
@pytest.mark.parametrize("precond", ["ilu0", "bjacobi"])
def test_lane_a_row_equals_four(precond, mixed):
    from paper_1711_10579_amd import binding as B

    ctx = B.pf_ctx_create(0)
    opt = dict(solver=B.PF_SOLVER_BICGSTAB, precision=B.PF_PREC_MIXED if mixed else B.PF_PREC_FP64, max_iter=40,
               precond=B.PF_PRECOND_ILU0 if precond == "ilu0" else B.PF_PRECOND_BJACOBI)
    small = [pfgen.make_polar_grid(2, 0, 0, 3), pfgen.make_polar_grid(3, 1, 1, 3, balanced=True), _star(41), _star(9),
             _mesh(40), _mesh(256), _mesh(257), _mesh(258)]
    grids = [_mesh(5000)] + small + [pfgen.perturb_loads(_mesh(40), i) for i in range(45)]
    rows = [g.n - 1 for g in grids]  # every bus but the slack
    assert -(-max(rows) // 256) * 256 * len(rows) - sum(rows) > 204800
    hs = [B.pf_create_from(ctx, g) for g in grids]
    print(f"{precond} mixed {mixed}: {len(hs)} grids", flush=True)
    res = B.pf_solve_batch(ctx, hs, **opt)
    for k, (h, b) in enumerate(zip(hs, res)):
        V = B.pf_get_voltage(h)
        if k < 12:
            r = B.pf_solve(h, **opt)
            assert (r.status, r.iters, r.linear_iters) == (b.status, b.iters, b.linear_iters), k
            assert np.array_equal(B.pf_get_voltage(h), V), k
        assert b.status == B.PF_CONVERGED, k
        h.close()
    ctx.close()
