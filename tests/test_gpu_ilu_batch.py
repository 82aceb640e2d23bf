"""GPU test of ILU(0) batches on the forms that only many instances take: the
factor of every instance in one launch, its levels of any width behind
barriers; and instances that sweep by levels beside the others' first part.
70 grids, one of whose first levels is wider than a factor launch's four
passes of targets; each is bit-identical to its solve alone.
"""

import numpy as np
import pytest

import pfgen

pytestmark = pytest.mark.gpu


def _mesh(n, seed=11):
    return pfgen.make_polar_grid(n, (3 * n) // 10, max(1, n // 10), seed, balanced=True)


@pytest.mark.parametrize("mixed", [False, True], ids=["fp64", "mixed"])
@pytest.mark.parametrize("solver", ["gmres", "bicgstab"])
def test_batch_equals_alone(solver, mixed):
    from paper_1711_10579_amd import binding as B

    ctx = B.pf_ctx_create(0)
    opt = dict(solver=B.PF_SOLVER_GMRES if solver == "gmres" else B.PF_SOLVER_BICGSTAB,
               precision=B.PF_PREC_MIXED if mixed else B.PF_PREC_FP64, max_iter=40)
    grids = [_mesh(9000), _mesh(2300), pfgen.make_feeder(900, 5), _mesh(2), _mesh(700)]
    grids += [pfgen.perturb_loads(_mesh(300), i) for i in range(65)]
    hs = [B.pf_create_from(ctx, g) for g in grids]
    print(f"{solver} mixed {mixed}", flush=True)
    res = B.pf_solve_batch(ctx, hs, **opt)
    for k, (h, b) in enumerate(zip(hs, res)):
        V = B.pf_get_voltage(h)
        assert b.status == B.PF_CONVERGED, k
        if k < 10:
            r = B.pf_solve(h, **opt)
            assert (r.status, r.iters, r.linear_iters) == (b.status, b.iters, b.linear_iters), k
            assert np.array_equal(B.pf_get_voltage(h), V), k
        h.close()
    ctx.close()


def test_parts_beside_large_level_sweeps():
    """A grid with a plan beside a feeder that sweeps by levels with its vector in
    more than 32 KB of LDS, the part then in a launch of its own."""
    from paper_1711_10579_amd import binding as B

    ctx = B.pf_ctx_create(0)
    opt = dict(solver=B.PF_SOLVER_BICGSTAB, max_iter=40)
    hs = [B.pf_create_from(ctx, g) for g in (_mesh(2300), pfgen.make_feeder(1200, 5))]
    parts = [B.pf_debug_sweep_check(h, B.PF_PREC_FP64)[2] for h in hs]
    assert min(parts[0]) >= 2 and parts[1] == (0, 0) and B.pf_case_info_get(hs[1])["n_unknown"] > 2048
    res = B.pf_solve_batch(ctx, hs, **opt)
    for h, b in zip(hs, res):
        V = B.pf_get_voltage(h)
        r = B.pf_solve(h, **opt)
        assert (r.status, r.iters, r.linear_iters) == (b.status, b.iters, b.linear_iters)
        assert b.status == B.PF_CONVERGED and np.array_equal(B.pf_get_voltage(h), V)
        h.close()
    ctx.close()
