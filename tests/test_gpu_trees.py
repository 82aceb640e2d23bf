"""GPU test of the upper levels of the sparse factor as subtrees (Sec. III-A
refactorisation and its backward solve, a case solved alone): shapes with one
column, levels of one row (a path) and of hundreds (a star's leaves, many to a
work-group's pass), lists longer than a group's four entries a lane, and a
mesh eliminated without a dense block, whose rows' blocks do not all fit in a
work-group's LDS.  The roots agree with the oracle within the parity tolerance
of 1e-7, and the same case in a batch (by levels) gives the same bits.
"""

import numpy as np
import pytest

import pfgen
from oracle import cim, polar

pytestmark = pytest.mark.gpu


def _radial(parents, seed=2):
    """Polar grid on the given tree (parent of bus k + 1), loads and line
    impedances so light that a path of all buses is an ordinary feeder."""
    import pins

    n = len(parents) + 1
    rng = np.random.default_rng(seed)
    b = np.arange(1, n)
    s = 0.2 / n
    return pins.polar_case(n, list(parents), list(b), [0.1 / n] * (n - 1), [0.3 / n] * (n - 1), [0.0] * (n - 1),
                           [3] + [1] * (n - 1), list(np.r_[0, -s * (0.5 + rng.random(n - 1))]),
                           list(np.r_[0, -0.4 * s * (0.5 + rng.random(n - 1))]), [1] * n)


SHAPES = [
    ("two", lambda: _radial([0]), {}),
    ("path600", lambda: _radial(range(599)), {}),
    ("star900", lambda: _radial([0] * 3 + [1 + k % 3 for k in range(896)]), {}),
    ("comb500", lambda: _radial([0 if k == 0 else k - 1 if k % 2 else k - 2 + (k == 2) for k in range(499)]), {}),
    ("mesh300", lambda: pfgen.make_polar_grid(300, 90, 30, 6, balanced=True), dict(dense_switch=1.0, min_dense=10000)),
    ("mesh900", lambda: pfgen.make_polar_grid(900, 270, 90, 6, balanced=True), dict(dense_switch=1.0, min_dense=10000)),
    ("mesh700wide", lambda: pfgen.make_polar_grid(700, 210, 70, 8, balanced=True), dict(lane_scale=4)),
    # the dense block's backward solve in one work-group, and a work-group a block
    ("mesh900single", lambda: pfgen.make_polar_grid(900, 270, 90, 6, balanced=True), dict(trsv_mode=2)),
    ("mesh900apart", lambda: pfgen.make_polar_grid(900, 270, 90, 6, balanced=True), dict(trsv_mode=1)),
    ("feeder400", lambda: pfgen.make_feeder(400, 3), {}),
]


@pytest.mark.parametrize("name,maker,sched", SHAPES, ids=[s[0] for s in SHAPES])
def test_alone_and_batched(name, maker, sched):
    from paper_1711_10579_amd import binding as B

    ctx = B.pf_ctx_create(0)
    g = maker()
    ref = (polar if hasattr(g, "bus_type") else cim).newton(g)
    h = [B.pf_create_from(ctx, g, schedule=B.pf_default_schedule(**sched)) for _ in range(2)]
    for precision in (B.PF_PREC_FP64, B.PF_PREC_MIXED):
        print(f"{name} precision {precision}", flush=True)
        r = B.pf_solve(h[0], precision=precision, max_iter=40)
        assert r.status == B.PF_CONVERGED, name
        V = B.pf_get_voltage(h[0])
        assert np.max(np.abs(V - ref.V)) <= 1e-7
        for q, c in zip(B.pf_solve_batch(ctx, h, precision=precision, max_iter=40), h):
            assert (q.status, q.iters, q.mismatch_inf) == (r.status, r.iters, r.mismatch_inf)
            assert np.array_equal(B.pf_get_voltage(c), V)
    for c in h:
        c.close()
    ctx.close()
