"""GPU test of the ILU(0) sweep lists' device memory, through a context with
allocator callbacks: a case whose lists get no memory sweeps by levels, also
when the refused allocation leaves an error behind in the HIP runtime; and every
byte a case has allocated is in pf_case_info's device_bytes or, for its launch
plans, in pf_case_plan_bytes.
"""

import ctypes

import numpy as np
import pytest

import pfgen
from oracle import polar

pytestmark = pytest.mark.gpu


def _hip():
    """The HIP runtime that the library uses in this process."""
    with open("/proc/self/maps") as f:
        path = next(l.split()[-1] for l in f if "libamdhip64.so" in l)
    return ctypes.CDLL(path)


def _context(B, refuse):
    """Context whose allocations go through hipMalloc, are recorded, and are
    refused by `refuse(index)`; a refusal follows a failed hipMalloc of 2^60
    bytes, as a refusal of the default allocator does."""
    hip = _hip()
    live, sizes = {}, []

    def alloc(nbytes, _user):
        p = ctypes.c_void_p()
        sizes.append(nbytes)
        if refuse(len(sizes) - 1):
            assert hip.hipMalloc(ctypes.byref(p), ctypes.c_size_t(1 << 60)) != 0
            return None
        assert hip.hipMalloc(ctypes.byref(p), ctypes.c_size_t(nbytes)) == 0
        live[p.value] = nbytes
        return p.value

    def free(ptr, _user):
        del live[ptr]
        assert hip.hipFree(ctypes.c_void_p(ptr)) == 0

    ctx = B.Context.__new__(B.Context)
    ctx._keep = [B.ALLOC_FN(alloc), B.FREE_FN(free)]
    ctx.handle = ctypes.c_void_p()
    assert B._lib.pf_ctx_create(0, None, *ctx._keep, None, ctypes.byref(ctx.handle)) == 0
    return ctx, live, sizes


def _mesh(n):
    return pfgen.make_polar_grid(n, (3 * n) // 10, n // 10, 11, balanced=True)


def test_lists_refused():
    from paper_1711_10579_amd import binding as B

    g = _mesh(2399)
    ref = polar.newton(g).V
    opt = dict(solver=B.PF_SOLVER_BICGSTAB, max_iter=40)
    lists = None
    for turn in ("granted", "refused"):
        ctx, live, sizes = _context(B, lambda k: turn == "refused" and k == lists)
        h = B.pf_create_from(ctx, g)
        # everything but the ILU(0) lists is there after a solve with the other preconditioner
        assert B.pf_solve(h, precond=B.PF_PRECOND_BJACOBI, **opt).status == B.PF_CONVERGED
        lists = len(sizes)
        print(turn, flush=True)
        for _ in range(2):
            assert B.pf_solve(h, precond=B.PF_PRECOND_ILU0, **opt).status == B.PF_CONVERGED
            assert np.max(np.abs(B.pf_get_voltage(h) - ref)) <= 1e-7
        assert len(sizes) == lists + 2  # the lists, the launch plan
        parts = B.pf_debug_sweep_check(h, B.PF_PREC_FP64)[2]
        assert (parts == (0, 0)) == (turn == "refused"), parts
        h.close()
        ctx.close()
        assert not live


@pytest.mark.parametrize("n", [300, 2399])
def test_every_byte_is_reported(n):
    from paper_1711_10579_amd import binding as B

    ctx, live, _ = _context(B, lambda k: False)
    h = B.pf_create_from(ctx, _mesh(n))

    def held():
        return B.pf_case_info_get(h)["device_bytes"] + B.pf_case_plan_bytes(h)

    assert B.pf_case_plan_bytes(h) == 0 and held() == sum(live.values())
    last = 0
    for opt in (dict(), dict(solver=B.PF_SOLVER_BICGSTAB, precond=B.PF_PRECOND_BJACOBI),
                dict(solver=B.PF_SOLVER_BICGSTAB, precond=B.PF_PRECOND_ILU0)):
        print(f"{n} buses, {opt}", flush=True)
        for _ in range(2):
            assert B.pf_solve(h, max_iter=40, **opt).status == B.PF_CONVERGED
            assert held() == sum(live.values())
        assert B.pf_case_plan_bytes(h) > last
        last = B.pf_case_plan_bytes(h)
    info = B.pf_case_info_get(h)
    assert info["device_bytes"] == info["resident_bytes"] + info["work_bytes"] + info["krylov_bytes"]
    h.close()
    assert not live
    ctx.close()
