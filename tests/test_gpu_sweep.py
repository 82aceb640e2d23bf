"""GPU test of the ILU(0) sweeps in parts (Sec. III-B preconditioner): Newton-
Krylov roots against the oracle, within the parity tolerance of 1e-7, on
graphs with no plan (a few nodes: levels), one part per sweep, several parts
with rows at the cap, and rows above it (the first level of a part); GMRES
(scaled input stored as basis vector) and BiCGStab, FP64 and FP32 inner
solves; the preconditioners in turn on one case (the entry values share the
block-Jacobi inverses' storage); and all of them as one batch, each instance
bit-identical to its solve alone.
"""

import sys

import numpy as np
import pytest

import pfgen
from oracle import cim, polar

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_1711_10579_amd import binding

    return binding


@pytest.fixture(scope="module")
def ctx(B):
    c = B.pf_ctx_create(0)
    yield c
    c.close()


def _mesh(n, seed=11):
    return pfgen.make_polar_grid(n, (3 * n) // 10, max(1, n // 10), seed, balanced=True)


MAKERS = [
    ("mesh2", lambda: pfgen.make_polar_grid(2, 0, 0, 3)),
    ("mesh3", lambda: pfgen.make_polar_grid(3, 1, 1, 3, balanced=True)),
    ("mesh33", lambda: _mesh(33)),
    ("mesh257", lambda: _mesh(257)),
    ("mesh2049", lambda: _mesh(2049)),
    ("tree300", lambda: pfgen.make_polar_grid(300, 0, 30, 7, balanced=True)),
    ("replica900", lambda: pfgen.replicate_polar(30, pfgen.BASE_SEED + 5)),
    ("feeder3", lambda: pfgen.make_feeder(3, 5)),
    ("feeder301", lambda: pfgen.make_feeder(301, 8)),
]


def _root(g):
    return (polar if hasattr(g, "bus_type") else cim).newton(g).V


@pytest.mark.parametrize("name,maker", MAKERS, ids=[m[0] for m in MAKERS])
def test_roots(B, ctx, name, maker):
    g = maker()
    ref = _root(g)
    h = B.pf_create_from(ctx, g)
    for solver in (B.PF_SOLVER_GMRES, B.PF_SOLVER_BICGSTAB):
        for prec in (B.PF_PREC_FP64, B.PF_PREC_MIXED):
            for pc in (B.PF_PRECOND_ILU0, B.PF_PRECOND_BJACOBI, B.PF_PRECOND_ILU0):
                print(f"{name} solver {solver} precision {prec} precond {pc}", flush=True)
                sys.stdout.flush()
                r = B.pf_solve(h, solver=solver, precision=prec, precond=pc, max_iter=40)
                assert r.status == B.PF_CONVERGED
                err = float(np.max(np.abs(B.pf_get_voltage(h) - ref)))
                assert err <= 1e-7, (name, solver, prec, pc, err)
    h.close()


@pytest.mark.parametrize("solver", ["gmres", "bicgstab"])
def test_batch_equals_alone(B, ctx, solver):
    sv = B.PF_SOLVER_GMRES if solver == "gmres" else B.PF_SOLVER_BICGSTAB
    hs = [B.pf_create_from(ctx, m()) for _, m in MAKERS]
    print(f"batch {solver}", flush=True)
    res = B.pf_solve_batch(ctx, hs, solver=sv, max_iter=40)
    got = [(r.status, r.iters, r.linear_iters, B.pf_get_voltage(h)) for r, h in zip(res, hs)]
    for (name, _), h, b in zip(MAKERS, hs, got):
        r = B.pf_solve(h, solver=sv, max_iter=40)
        assert (r.status, r.iters, r.linear_iters) == b[:3], name
        assert np.array_equal(B.pf_get_voltage(h), b[3]), name
        h.close()
