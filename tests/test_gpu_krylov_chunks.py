"""GPU test of the Krylov kernels' forms for batches of unequal and of small
grids: chunks by a list (more than 256 work-groups of the grid without one), and
BiCGStab's matrix products with a lane a row (room for more than 65,536 rows
past the instances' own): a large grid beside small ones, and very many small
ones, with rows of one to forty blocks (a star's middle) and instances of one
row to a whole chunk of 256 and one more.  The grids alone take neither form;
every result is bit-identical to its solve alone.
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


def _check(maker, **opt):
    from paper_1711_10579_amd import binding as B

    opt = dict(opt, max_iter=40)
    ctx = B.pf_ctx_create(0)
    small = [pfgen.make_polar_grid(2, 0, 0, 3), pfgen.make_polar_grid(3, 1, 1, 3, balanced=True), _star(41), _star(9),
             _mesh(40), _mesh(256), _mesh(257), _mesh(258)]
    grids = maker(small)
    rows = [g.n - 1 for g in grids]  # every bus but the slack
    hs = [B.pf_create_from(ctx, g) for g in grids]
    res = B.pf_solve_batch(ctx, hs, **opt)
    for k, (h, b) in enumerate(zip(hs, res)):
        assert b.status == B.PF_CONVERGED, k
        if k < 12:
            V = B.pf_get_voltage(h)
            r = B.pf_solve(h, **opt)
            assert (r.status, r.iters, r.linear_iters) == (b.status, b.iters, b.linear_iters), k
            assert np.array_equal(B.pf_get_voltage(h), V), k
        h.close()
    ctx.close()
    return rows


@pytest.mark.parametrize("mixed", [0, 1], ids=["fp64", "mixed"])
@pytest.mark.parametrize("precond", [0, 1], ids=["ilu0", "bjacobi"])
@pytest.mark.parametrize("solver", [1, 2], ids=["gmres", "bicgstab"])
def test_chunks_by_a_list(solver, precond, mixed):
    print(f"solver {solver} precond {precond} mixed {mixed}", flush=True)
    rows = _check(lambda small: small + [_mesh(5000)] + [pfgen.perturb_loads(_mesh(40), i) for i in range(45)],
                  solver=solver, precond=precond, precision=mixed)
    chunks = [-(-r // 256) for r in rows]
    assert max(chunks) * len(chunks) - sum(chunks) > 256


@pytest.mark.parametrize("mixed", [0, 1], ids=["fp64", "mixed"])
def test_lane_a_row(mixed):
    print(f"mixed {mixed}", flush=True)
    base = _mesh(40)
    rows = _check(lambda small: small + [pfgen.perturb_loads(base, i) for i in range(320)], solver=2, precond=1,
                  precision=mixed)
    assert sum(-(-r // 256) * 256 - r for r in rows) > 65536
