"""GPU test of the ILU(0) sweeps in parts (Sec. III-B preconditioner) on grids
that get a plan, asserted through the number of parts: an application against
the triangular solves in FP64 from the same factor.  In FP64 the difference
stays at rounding: some 30 chained 2x2 products of values around one, at
1.1e-16 each and with the triangles' condition (hundreds) below 1e-11.  With an
FP32 factor and FP32 vectors it is no larger than that of sweeps by levels,
whose rows are summed in FP64 and stored in FP32.
"""

import pytest

import pfgen

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
