"""GPU test of the dense trailing block's step launches (Sec. III-A): grids
eliminated as one dense block, at orders around the 64-wide steps (a partial,
a full and a barely started last step, one to ten steps), so that tiles take
one step's update or two at a time; alone (a work-group per quarter of a row
tile) and in batches with more panel work-groups than CUs (a work-group per
row tile).  The roots agree with the oracle within the parity tolerance of
1e-7, and every instance of a batch is bit-identical to its solve alone.
"""

import numpy as np
import pytest

import pfgen
from oracle import polar

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


# buses, seed, nodes of the dense block (half its order)
GRIDS = [(33, 1, 31), (34, 1, 32), (35, 5, 33), (66, 5, 63), (65, 1, 64), (67, 5, 65), (98, 5, 96), (132, 5, 129),
         (162, 5, 160), (226, 5, 224), (310, 5, 309)]


@pytest.mark.parametrize("precision", [0, 1], ids=["fp64", "mixed"])
def test_dense_orders(B, ctx, precision):
    sc = B.pf_default_schedule(dense_switch=1e-6, min_dense=1)
    opts = dict(precision=precision, max_iter=40)
    hs, alone = [], []
    for n, seed, nd in GRIDS:
        g = pfgen.make_polar_grid(n, (3 * n) // 10, n // 10, seed, balanced=True)
        ref = polar.newton(g).V
        for copy in range(3 if n < 200 else 7):
            f = 1.0 - 0.03 * copy
            h = B.pf_create_from(ctx, g.with_injections(g.p_sp * f, g.q_sp * f), schedule=sc)
            print(f"order {2 * nd} copy {copy} precision {precision}", flush=True)
            r = B.pf_solve(h, **opts)
            assert r.status == B.PF_CONVERGED, n
            V = B.pf_get_voltage(h)
            if copy == 0:
                assert B.pf_case_info_get(h)["n_dense"] == nd
                assert np.max(np.abs(V - ref)) <= 1e-7, n
            hs.append(h)
            alone.append((r.status, r.iters, r.mismatch_inf, V))
    print("batch", flush=True)
    for r, h, a in zip(B.pf_solve_batch(ctx, hs, **opts), hs, alone):
        assert (r.status, r.iters, r.mismatch_inf) == a[:3]
        assert np.array_equal(B.pf_get_voltage(h), a[3])
    for h in hs:
        h.close()
