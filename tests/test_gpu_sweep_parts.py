"""GPU test of the ILU(0) sweeps in parts (Sec. III-B preconditioner) on grids
that get a plan, asserted through the number of parts: an application against
the triangular solves in FP64 from the same factor.  In FP64 the difference
stays at rounding: some 30 chained 2x2 products of values around one, at
1.1e-16 each and with the triangles' condition (hundreds) below 1e-11.  With an
FP32 factor and FP32 vectors it is no larger than that of sweeps by levels,
whose rows are summed in FP64 and stored in FP32.  Then whole Newton-Krylov
solves of such grids: roots against the oracle within the parity tolerance of
1e-7, the preconditioners in turn on one case (the entry values share the
block-Jacobi inverses' storage), and batches of grids with different numbers of
parts beside ones that sweep by levels, each bit-identical to its solve alone.
"""

import numpy as np
import pytest

import pfgen
from oracle import cim, polar

pytestmark = pytest.mark.gpu


def _mesh(n, seed=11):
    return pfgen.make_polar_grid(n, (3 * n) // 10, max(1, n // 10), seed, balanced=True)


PLANNED = [
    ("mesh2050", lambda: _mesh(2050)),
    ("mesh2399", lambda: _mesh(2399)),
    ("mesh4000", lambda: _mesh(4000)),
    ("replica80", lambda: pfgen.replicate_polar(80, pfgen.BASE_SEED + 5)),
    ("mesh10000", lambda: _mesh(10000)),
]


@pytest.mark.parametrize("name,maker", PLANNED, ids=[m[0] for m in PLANNED])
def test_application(name, maker):
    from paper_1711_10579_amd import binding as B

    ctx = B.pf_ctx_create(0)
    h = B.pf_create_from(ctx, maker())
    for precision in (B.PF_PREC_FP64, B.PF_PREC_MIXED):
        dev, lev, parts = B.pf_debug_sweep_check(h, precision, seed=7)
        print(f"{name} precision {precision}: parts {parts}, deviation {dev:.3g}, by levels {lev:.3g}", flush=True)
        assert min(parts) >= 2
        assert dev <= (1e-11 if precision == B.PF_PREC_FP64 else lev)
    h.close()
    ctx.close()


SOLVERS = ["gmres", "bicgstab"]


def _solver(B, name):
    return B.PF_SOLVER_GMRES if name == "gmres" else B.PF_SOLVER_BICGSTAB


@pytest.mark.parametrize("name,maker", PLANNED[:4], ids=[m[0] for m in PLANNED[:4]])
def test_roots(name, maker):
    from paper_1711_10579_amd import binding as B

    ctx = B.pf_ctx_create(0)
    g = maker()
    ref = polar.newton(g).V
    h = B.pf_create_from(ctx, g)
    assert min(B.pf_debug_sweep_check(h, B.PF_PREC_FP64)[2]) >= 2
    for solver in SOLVERS:
        for prec in (B.PF_PREC_FP64, B.PF_PREC_MIXED):
            for pc in (B.PF_PRECOND_ILU0, B.PF_PRECOND_BJACOBI, B.PF_PRECOND_ILU0):
                print(f"{name} {solver} precision {prec} precond {pc}", flush=True)
                r = B.pf_solve(h, solver=_solver(B, solver), precision=prec, precond=pc, max_iter=40)
                assert r.status == B.PF_CONVERGED
                assert np.max(np.abs(B.pf_get_voltage(h) - ref)) <= 1e-7
    h.close()
    ctx.close()


# grids of one part count beside another's, of few rows (their last work-group
# is mostly padding), and ones without a plan
BATCH = [
    ("mesh33", lambda: _mesh(33), False),
    ("mesh2050", lambda: _mesh(2050), True),
    ("mesh4000", lambda: _mesh(4000), True),
    ("feeder301", lambda: pfgen.make_feeder(301, 8), False),
    ("mesh2399", lambda: _mesh(2399, 5), True),
    ("mesh1500", lambda: _mesh(1500), False),
    ("replica80", lambda: pfgen.replicate_polar(80, pfgen.BASE_SEED + 5), True),
]


@pytest.mark.parametrize("mixed", [False, True], ids=["fp64", "mixed"])
@pytest.mark.parametrize("solver", SOLVERS)
def test_batch_equals_alone(solver, mixed):
    from paper_1711_10579_amd import binding as B

    ctx = B.pf_ctx_create(0)
    opt = dict(solver=_solver(B, solver), precision=B.PF_PREC_MIXED if mixed else B.PF_PREC_FP64, max_iter=40)
    grids = [m() for _, m, _ in BATCH]
    hs = [B.pf_create_from(ctx, g) for g in grids]
    parts = [B.pf_debug_sweep_check(h, opt["precision"])[2] for h in hs]
    print(f"{solver} mixed {mixed}: parts {parts}", flush=True)
    assert [min(p) >= 2 for p in parts] == [planned for _, _, planned in BATCH]
    assert len({p for p in parts if min(p)}) >= 2
    res = B.pf_solve_batch(ctx, hs, **opt)
    got = [(r.status, r.iters, r.linear_iters, B.pf_get_voltage(h)) for r, h in zip(res, hs)]
    for (name, _, _), g, h, b in zip(BATCH, grids, hs, got):
        r = B.pf_solve(h, **opt)
        assert (r.status, r.iters, r.linear_iters) == b[:3] and r.status == B.PF_CONVERGED, name
        assert np.array_equal(B.pf_get_voltage(h), b[3]), name
        ref = (polar if hasattr(g, "bus_type") else cim).newton(g).V
        assert np.max(np.abs(b[3] - ref)) <= 1e-7, name
        h.close()
    ctx.close()
