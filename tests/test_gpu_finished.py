"""GPU test that the finished instances of a batch cost next to nothing: with
one feeder at a flat start and the others at their roots, the launches of the
Jacobian fill and of the sparse refactorisation take less than 0.6 of what
they take with every feeder at a flat start.  The finished instances'
work-groups read an item, a descriptor and at most one entry more, so what
remains is a launch, some 3 us, and one feeder's chain; the feeders are so many
that the launches of all take several times that.  The same for the ILU(0)
sweeps in parts of a Newton-Krylov batch.
"""

import numpy as np
import pytest

import pfgen

pytestmark = pytest.mark.gpu


def _flat(g):
    return np.where(g.node_type == pfgen.PQ, 1.0, g.v_mag) * np.exp(1j * g.v_ang)


def test_finished_instances_leave():
    from paper_1711_10579_amd import binding as B

    ctx = B.pf_ctx_create(0)
    g = pfgen.make_feeder(900, 4)
    hs = [B.pf_create_from(ctx, pfgen.perturb_loads(g, i)) for i in range(160)]
    classes = ("PF_K_JFILL", "PF_K_SPARSE_FACTOR")

    def per_launch(flat):
        """ms a launch of each class, of the second of two equal solves."""
        for _ in range(2):
            for h in hs if flat else hs[:1]:
                B.pf_set_voltage(h, _flat(g))
            B.pf_profile_reset(ctx)
            res = B.pf_solve_batch(ctx, hs, flat_start=0)
        assert all(r.status == B.PF_CONVERGED for r in res)
        assert res[0].iters > 0 and all((r.iters > 0) == flat for r in res[1:])
        st = [B.pf_kernel_stats(ctx, getattr(B, k)) for k in classes]
        return [s["ms"] / s["launches"] for s in st]

    B.pf_profile_enable(ctx, sum(1 << getattr(B, k) for k in classes))
    every, one = per_launch(True), per_launch(False)
    B.pf_profile_enable(ctx, 0)
    for k, a, b in zip(classes, every, one):
        print(f"{k}: all {1e3 * a:.1f} us a launch, one {1e3 * b:.1f}", flush=True)
    for k, a, b in zip(classes, every, one):
        assert b < 0.6 * a, (k, a, b)
    for h in hs:
        h.close()
    ctx.close()


@pytest.mark.parametrize("solver", ["gmres", "bicgstab"])
def test_finished_instances_leave_the_sweeps(solver):
    from paper_1711_10579_amd import binding as B

    ctx = B.pf_ctx_create(0)
    g = pfgen.make_polar_grid(3000, 900, 300, 11, balanced=True)
    hs = [B.pf_create_from(ctx, pfgen.perturb_loads(g, i)) for i in range(160)]
    sv = B.PF_SOLVER_GMRES if solver == "gmres" else B.PF_SOLVER_BICGSTAB

    def per_application(flat):
        for _ in range(2):
            for h in hs if flat else hs[:1]:
                B.pf_set_voltage(h, np.ones(g.n, complex))
            B.pf_profile_reset(ctx)
            res = B.pf_solve_batch(ctx, hs, flat_start=0, solver=sv, max_iter=40)
        assert all(r.status == B.PF_CONVERGED for r in res)
        assert res[0].iters > 0 and all((r.iters > 0) == flat for r in res[1:])
        s = B.pf_kernel_stats(ctx, B.PF_K_PRECOND_APPLY)
        return s["ms"] / s["launches"]

    B.pf_profile_enable(ctx, 1 << B.PF_K_PRECOND_APPLY)
    every, one = per_application(True), per_application(False)
    B.pf_profile_enable(ctx, 0)
    print(f"{solver}: all {1e3 * every:.1f} us an application, one {1e3 * one:.1f}", flush=True)
    assert one < 0.6 * every, (every, one)
    for h in hs:
        h.close()
    ctx.close()
