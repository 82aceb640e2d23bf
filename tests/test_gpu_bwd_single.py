"""GPU test of the dense blocks' backward solve in one work-group per instance
(Sec. III-A triangular solve): a batch of more dense blocks than the automatic
choice runs apart, and one that asks for that form, at orders around the
64-row blocks; every grid's voltages are bit-identical to its solve alone,
where the blocks run apart, and within the parity tolerance of 1e-7 of the
oracle.
"""

import numpy as np
import pytest

import pfgen
from oracle import polar

pytestmark = pytest.mark.gpu

# every node in the dense block
ALL_DENSE = dict(dense_switch=1e-9, min_dense=1)


@pytest.mark.parametrize("n,count,sched", [
    (500, 200, dict(ALL_DENSE)),  # 200 x 16 blocks > 3,072
    (33, 3, dict(ALL_DENSE, trsv_mode=2)),  # order 62: one block
    (34, 3, dict(ALL_DENSE, trsv_mode=2)),  # order 66
    (97, 3, dict(ALL_DENSE, trsv_mode=2)),  # order 190
    (1200, 3, dict(trsv_mode=2)),
], ids=["automatic", "order62", "order66", "order190", "mesh1200"])
def test_single_equals_apart(n, count, sched):
    from paper_1711_10579_amd import binding as B

    ctx = B.pf_ctx_create(0)
    g = pfgen.make_polar_grid(n, (3 * n) // 10, n // 10, 17, balanced=True)
    grids = [pfgen.perturb_loads(g, i) for i in range(count)]
    hs = [B.pf_create_from(ctx, c, schedule=B.pf_default_schedule(**sched)) for c in grids]
    order = 2 * B.pf_case_info_get(hs[0])["n_dense"]
    blocks = count * ((order + 63) // 64)
    print(f"order {order}, {blocks} blocks", flush=True)
    assert blocks > 3072 or sched.get("trsv_mode") == 2
    apart = [B.pf_create_from(ctx, c, schedule=B.pf_default_schedule(**dict(sched, trsv_mode=1))) for c in grids[:3]]
    for precision in (B.PF_PREC_FP64, B.PF_PREC_MIXED):
        res = B.pf_solve_batch(ctx, hs, precision=precision, max_iter=40)
        assert all(r.status == B.PF_CONVERGED for r in res)
        for c, h, a in zip(grids, hs, apart):
            V = B.pf_get_voltage(h)
            assert B.pf_solve(a, precision=precision, max_iter=40).status == B.PF_CONVERGED
            assert np.array_equal(B.pf_get_voltage(a), V)
            assert np.max(np.abs(V - polar.newton(c).V)) <= 1e-7
    for h in hs + apart:
        h.close()
    ctx.close()
