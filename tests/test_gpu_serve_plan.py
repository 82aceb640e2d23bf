"""GPU test that pf_submit plans a case's ILU(0) sweeps without holding up the
requests in flight: small requests submitted just before a large Newton-Krylov
one run while that call makes its plans.
"""

import time

import pytest

import pfgen

pytestmark = pytest.mark.gpu


def test_requests_run_during_a_plan():
    from paper_1711_10579_amd import binding as B

    ctx = B.pf_ctx_create(0)
    B.pf_serve_config(ctx, max_bytes=0, max_slots=4)
    grid = pfgen.config_case(0)
    small = [B.pf_create_from(ctx, pfgen.perturb_loads(grid, i)) for i in range(12)]
    g = pfgen.replicate_polar(1600, pfgen.BASE_SEED + 5)

    def wait(tickets):
        out = {}
        while len(out) < len(tickets):
            for t in tickets:
                if t not in out:
                    done, r = B.pf_poll(ctx, t)
                    if done:
                        out[t] = r
        return [out[t] for t in tickets]

    assert all(r.status == B.PF_CONVERGED for r in wait([B.pf_submit(ctx, h) for h in small]))
    a = time.perf_counter()
    assert all(r.status == B.PF_CONVERGED for r in wait([B.pf_submit(ctx, h) for h in small]))
    alone = time.perf_counter() - a
    for turn in range(3):
        # a case of its own each turn: its plans are made by its first request;
        # its launch plan is there (the block-Jacobi request), which is made
        # under the lock
        large = B.pf_create_from(ctx, g)
        opts = dict(solver=B.PF_SOLVER_BICGSTAB, max_iter=40)
        assert wait([B.pf_submit(ctx, large, precond=B.PF_PRECOND_BJACOBI, **opts)])[0].status == B.PF_CONVERGED
        print(f"turn {turn}", flush=True)
        tickets = [B.pf_submit(ctx, h) for h in small]
        a = time.perf_counter()
        last = B.pf_submit(ctx, large, precond=B.PF_PRECOND_ILU0, **opts)
        took = time.perf_counter() - a
        polled = [B.pf_poll(ctx, t) for t in tickets]
        done = sum(d for d, _ in polled)
        print(f"12 requests take {1e3 * alone:.2f} ms; {done} done after a pf_submit of {1e3 * took:.2f} ms", flush=True)
        wait([t for t, (d, _) in zip(tickets, polled) if not d])
        assert wait([last])[0].status == B.PF_CONVERGED
        large.close()
        # the plans take several times as long as these requests
        if took > 3 * alone:
            break
    else:
        pytest.skip("the small requests took longer than the plans")
    assert done >= 6
    for h in small:
        h.close()
    ctx.close()
