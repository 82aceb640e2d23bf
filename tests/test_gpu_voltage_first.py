"""GPU test that reading voltages allocates nothing: the first pf_get_voltage
of a context succeeds while a HIP graph of the caller is being captured in the
global mode, which refuses allocations, and leaves that capture intact; and that a
context without pinned memory reads the same.  The values are the ones that
were set.
"""

import numpy as np
import pytest

import pfgen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [30, 40000])
def test_first_read_during_a_capture(n):
    import torch

    from paper_1711_10579_amd import binding as B

    ctx = B.pf_ctx_create(0)
    h = B.pf_create_from(ctx, pfgen.make_polar_grid(n, 0, 0, 4, balanced=True))
    V = 1.0 + 0.1 * np.random.default_rng(n).standard_normal(n) + 0.2j
    B.pf_set_voltage(h, V)
    x = torch.ones(64, device="cuda")
    graph = torch.cuda.CUDAGraph()
    print(f"{n} nodes", flush=True)
    with torch.cuda.graph(graph, capture_error_mode="global"):
        y = 3 * x
        got = B.pf_get_voltage(h)
    assert np.array_equal(got, V)
    for k in range(3):
        x.fill_(k)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, torch.full_like(y, 3 * k))
        assert np.array_equal(B.pf_get_voltage(h), V)
    h.close()
    ctx.close()


@pytest.mark.parametrize("n", [2, 1025, 40000])
def test_without_pinned_memory(n):
    from paper_1711_10579_amd import binding as B

    ctx = B.pf_ctx_create(0)
    h = B.pf_create_from(ctx, pfgen.make_polar_grid(n, 0, 0, 4, balanced=True))
    V = 1.0 + 0.1 * np.random.default_rng(n).standard_normal(n) + 0.2j
    B.pf_set_voltage(h, V)
    assert np.array_equal(B.pf_get_voltage(h), V)
    B.pf_debug_drop_pinned(ctx)
    for _ in range(2):
        assert np.array_equal(B.pf_get_voltage(h), V)
    h.close()
    ctx.close()
