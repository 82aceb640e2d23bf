"""GPU test of reading voltages back (pf_get_voltage): values set on a case
come back bit for bit, at sizes around the blocks (1,024 nodes) and pinned
halves (32,768 nodes) the read goes through, two cases in turn (each read
overwrites the other's staged values), and after a solve.
"""

import numpy as np
import pytest

import pfgen
from oracle import polar

pytestmark = pytest.mark.gpu


def test_round_trip():
    from paper_1711_10579_amd import binding as B

    ctx = B.pf_ctx_create(0)
    rng = np.random.default_rng(3)
    hs = []
    for n in (2, 1023, 1024, 1025, 2049, 32768, 32769, 66561):
        print(f"nodes {n}", flush=True)
        h = B.pf_create_from(ctx, pfgen.make_polar_grid(n, 0, 0, 4, balanced=True))
        V = 1.0 + 0.1 * (rng.standard_normal(n) + 1j * rng.standard_normal(n))
        B.pf_set_voltage(h, V)
        hs.append((h, V))
        for g, U in hs[-2:] * 2:
            assert np.array_equal(B.pf_get_voltage(g), U), (n, len(U))
    for h, _ in hs:
        h.close()
    g = pfgen.make_polar_grid(1100, 330, 110, 9, balanced=True)
    h = B.pf_create_from(ctx, g)
    assert B.pf_solve(h).status == B.PF_CONVERGED
    assert np.max(np.abs(B.pf_get_voltage(h) - polar.newton(g).V)) <= 1e-7
    h.close()
    ctx.close()
