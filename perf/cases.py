"""Performance cases of the power-flow library: what they run and on which inputs.

Every case goes through the public entry points of the ctypes binding, as a
program that solves power flows calls them: a grid is created once
(``pf_create``), the day's loads come in with the case, a pass solves it
(``pf_solve``, ``pf_solve_batch`` or ``pf_submit`` / ``pf_poll``) from a flat
start and reads the voltages back (``pf_get_voltage``).  The grids are the
seeded ones of ``pfgen`` at the sizes of this repository's benchmark and
tests; the topology belongs to the case, the loads (a factor per bus around
the grid's own) to the seed.

Fields of a case:
  what     "solve" one grid at a time, "batch" one pf_solve_batch, "serve" all
           requests submitted at once and polled until done
  grid     "meshed" (tree with 0.3 n chords, 10 % PV), "grid30" (the 30-bus
           grid), "replica" (copies of the 30-bus block), "feeder" (a
           three-phase radial feeder), "feeders" (copies of the 906-bus
           feeder), "scenarios" (grids of log-uniform sizes), "pool" (meshed
           grids and feeders of a serving pool)
  size     buses, blocks, copies, or the largest grid of a mix
  count    grids of a batch or requests of a serving pass
  grid_seed  seed of the topology
  solver   "lu", "gmres", "bicgstab"; precond "ilu0" or "bjacobi"
  mixed    FP32 factor and inner solves (FP64 mismatch, update and test)
  tol      stop tolerance on the FP64 mismatch.  LU takes the default 1e-8
           (its last step is quadratic, the voltages are the root to
           rounding); inexact inner solves stop at 1e-11 and mixed precision
           at 1e-10, so that the voltages do not depend on where the last
           inexact step happened to land
"""

import functools
import heapq
import math

import numpy as np

import pfgen
from paper_1711_10579_amd import binding as B

SOLVERS = {"lu": B.PF_SOLVER_LU, "gmres": B.PF_SOLVER_GMRES, "bicgstab": B.PF_SOLVER_BICGSTAB}
PRECONDS = {"ilu0": B.PF_PRECOND_ILU0, "bjacobi": B.PF_PRECOND_BJACOBI}


def _case(name, what, grid, size, grid_seed, count=1, solver="lu", precond="ilu0", mixed=False, tol=None):
    if tol is None:
        tol = 1e-11 if solver != "lu" else 1e-10 if mixed else 1e-8
    c = {"what": what, "grid": grid, "size": size, "grid_seed": grid_seed, "count": count, "solver": solver,
         "precond": precond, "mixed": mixed, "tol": tol}
    return {"name": name, **c} if name else c


def listed():
    return [
        # the smallest call: one 30-bus grid, where launches and the host path count
        _case("grid30_lu", "solve", "grid30", 30, pfgen.BASE_SEED),
        # one distribution feeder of 907 buses (2,462 phase-nodes): an ordinary
        # three-phase study, shallow dense work, many small levels
        _case("feeder907_lu", "solve", "feeders", 1, pfgen.BASE_SEED + 6),
        # the benchmark's headline: one 10,000-bus transmission grid
        _case("grid10k_lu", "solve", "meshed", 10000, pfgen.BASE_SEED + 1),
        # 16 load scenarios of that grid in one batch (day-ahead scenarios)
        _case("grid10k_batch16_lu", "batch", "meshed", 10000, pfgen.BASE_SEED + 1, count=16),
        # Newton-Krylov on that grid with the default preconditioner: the
        # method the reference tests and the restarted one
        _case("grid10k_gmres_ilu0", "solve", "meshed", 10000, pfgen.BASE_SEED + 1, solver="gmres"),
        _case("grid10k_bicgstab_ilu0", "solve", "meshed", 10000, pfgen.BASE_SEED + 1, solver="bicgstab"),
        # contingency-style batch: 512 grids of 100-5,000 buses, each its own
        # topology, FP32 inner solves
        _case("scenarios512_mixed", "batch", "scenarios", 5000, pfgen.BASE_SEED + 3, count=512, mixed=True),
        # a serving burst: 48 requests on a pool of 1,000-20,000-bus grids and
        # 500-3,000-bus feeders, under a 2 GiB pool budget, FP32 inner solves
        _case("served48_mixed", "serve", "pool", 20000, pfgen.BASE_SEED + 4, count=48, mixed=True),
        # the replicated 48,000-bus grid: direct, and Newton-Krylov with either
        # preconditioner (its ILU(0) levels are too wide for one work-group)
        _case("rep48k_lu", "solve", "replica", 1600, pfgen.BASE_SEED + 5),
        _case("rep48k_bicgstab_bjacobi", "solve", "replica", 1600, pfgen.BASE_SEED + 5, solver="bicgstab",
              precond="bjacobi"),
        _case("rep48k_bicgstab_ilu0", "solve", "replica", 1600, pfgen.BASE_SEED + 5, solver="bicgstab"),
        # the largest: 256 copies of the feeder, 231,682 buses, 628,742
        # phase-nodes (its mismatch cannot be certified below 2e-8 in FP64)
        _case("feeder231k_lu", "solve", "feeders", 256, pfgen.BASE_SEED + 6, tol=1e-7),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges: the sizes of the listed ones and all between."""
    kind = rng.choice(["mesh_lu", "mesh_lu", "feeder_lu", "feeders_lu", "replica_lu", "mesh_krylov", "mesh_krylov",
                       "replica_krylov", "batch", "scenarios", "pool"])
    gs = pfgen.BASE_SEED + rng.randrange(1000, 1000000)
    solver, precond = rng.choice(["gmres", "bicgstab"]), rng.choice(["ilu0", "bjacobi"])
    if kind == "mesh_lu":
        return _case(None, "solve", "meshed", _log_int(rng, 31, 20000), gs, mixed=rng.random() < 0.5)
    if kind == "feeder_lu":
        return _case(None, "solve", "feeder", _log_int(rng, 30, 3000), gs, mixed=rng.random() < 0.5)
    if kind == "feeders_lu":
        return _case(None, "solve", "feeders", _log_int(rng, 2, 128), pfgen.BASE_SEED + 6)
    if kind == "replica_lu":
        return _case(None, "solve", "replica", _log_int(rng, 3, 1599), pfgen.BASE_SEED + 5)
    if kind == "mesh_krylov":
        return _case(None, "solve", "meshed", _log_int(rng, 31, 9999), gs, solver=solver, precond=precond)
    if kind == "replica_krylov":
        return _case(None, "solve", "replica", _log_int(rng, 3, 1599), pfgen.BASE_SEED + 5, solver="bicgstab",
                     precond=precond)
    if kind == "batch":
        return _case(None, "batch", "meshed", _log_int(rng, 31, 9999), gs, count=rng.randrange(2, 17))
    if kind == "scenarios":
        return _case(None, "batch", "scenarios", _log_int(rng, 150, 5000), gs, count=_log_int(rng, 8, 400), mixed=True)
    return _case(None, "serve", "pool", _log_int(rng, 2000, 20000), gs, count=rng.randrange(5, 48), mixed=True)


# ---------------------------------------------------------------------------
# grids


def _meshed(n, seed):
    return pfgen.make_polar_grid(n, (3 * n) // 10, max(1, n // 10), seed, balanced=True)


@functools.lru_cache(maxsize=8)
def _grids(grid, size, grid_seed, count):
    """The topologies of a case with their base loads (one grid, unless it is a mix)."""
    if grid == "grid30":
        return [pfgen.config_case(0, grid_seed)]
    if grid == "meshed":
        return [_meshed(size, grid_seed)]
    if grid == "replica":
        return [pfgen.replicate_polar(size, grid_seed)]
    if grid == "feeder":
        return [pfgen.make_feeder(size, grid_seed)]
    if grid == "feeders":
        return [pfgen.replicate_feeder(size, grid_seed)]
    rng = np.random.default_rng(grid_seed)

    def sizes(lo, hi, k):
        return np.exp(rng.uniform(math.log(lo), math.log(hi), k)).round().astype(int)

    if grid == "scenarios":
        return [_meshed(int(n), grid_seed + 1 + i) for i, n in enumerate(sizes(100, size, count))]
    feeders = count // 3
    out = [_meshed(int(n), grid_seed + 1 + i) for i, n in enumerate(sizes(1000, size, count - feeders))]
    return out + [pfgen.make_feeder(int(n), grid_seed + 501 + i) for i, n in enumerate(rng.integers(500, 3001, feeders))]


def _grid_args(case):
    return case["grid"], case["size"], case["grid_seed"], case["count"]


def _inputs(case, seed):
    """The grids with the seed's loads: every load times U[0.8, 1.2] (the
    replicated transmission grid, which one slack bus serves, U[0.98, 1.02])."""
    base = _grids(*_grid_args(case))
    base = base * case["count"] if len(base) == 1 else base
    w = 0.02 if case["grid"] == "replica" else 0.2
    return [pfgen.perturb_loads(g, seed * 1009 + i, 1 - w, 1 + w) for i, g in enumerate(base)]


# ---------------------------------------------------------------------------
# one pass


@functools.lru_cache(maxsize=1)
def _context():
    return B.pf_ctx_create(0)


def prepare(case, seed):
    ctx = _context()
    if case["what"] == "serve":
        ctx = B.pf_ctx_create(0)
        B.pf_serve_config(ctx, max_bytes=2 << 30)
    opts = B.pf_default_options(solver=SOLVERS[case["solver"]], precond=PRECONDS[case["precond"]],
                                precision=B.PF_PREC_MIXED if case["mixed"] else B.PF_PREC_FP64, tol=case["tol"],
                                max_iter=40)
    handles = [B.pf_create_from(ctx, g) for g in _inputs(case, seed)]
    return {"what": case["what"], "concat": case["count"] > 60, "ctx": ctx, "handles": handles, "opts": opts}


def run(state):
    hs, opts = state["handles"], state["opts"]
    if state["what"] == "solve":
        res = [B.pf_solve(hs[0], opts)]
    elif state["what"] == "batch":
        res = B.pf_solve_batch(state["ctx"], hs, opts)
    else:
        tickets = [B.pf_submit(state["ctx"], h, opts) for h in hs]
        res = []
        for t in tickets:
            done = False
            while not done:
                done, r = B.pf_poll(state["ctx"], t)
            res.append(r)
    status = np.array([r.status for r in res], np.int32)
    V = [B.pf_get_voltage(h) for h in hs]
    return {"status": status, "V": np.concatenate(V) if state["concat"] else V}


# ---------------------------------------------------------------------------
# what a pass cannot do without


def work(case):
    """Bytes: the Ybus (column index and complex value per entry), the row
    pointers, the set-points and the voltages.  Flops: per Newton step the
    mismatch (8 per Ybus entry) and the Jacobian's 2x2 block per entry with
    its share of the solve (at least 16), over 4 steps (2 on a feeder)."""
    nbytes = flops = 0
    base = _grids(*_grid_args(case))
    for g in base:
        polar = hasattr(g, "bus_type")
        nbytes += 20 * g.nnz + g.n * (4 + 1 + 32 + (0 if polar else 48) + 16)
        flops += (4 if polar else 2) * 24 * g.nnz
    k = case["count"] if len(base) == 1 else 1
    return {"bytes": k * nbytes, "flops": k * flops}


# ---------------------------------------------------------------------------
# the root in 64 bits: Newton's method on the power balance in rectangular
# coordinates, each step a 2x2-block elimination by smallest degree with a
# dense solve of what remains


def _solve_blocks(nodes, rows, rhs):
    """rows[i][j]: 2x2 blocks (a, b, c, d) of a structurally symmetric matrix
    over `nodes`, rhs[i]: pairs; both are consumed.  Returns {i: (x0, x1)}."""
    heap = [(len(rows[i]), i) for i in nodes]
    heapq.heapify(heap)
    left, done = set(nodes), []
    while left:
        deg, i = heapq.heappop(heap)
        if i not in left:
            continue
        if deg != len(rows[i]):
            heapq.heappush(heap, (len(rows[i]), i))
            continue
        if len(left) <= 1200 and deg > 0.1 * len(left):
            break
        left.remove(i)
        done.append(i)
        ri = rows[i]
        a, b, c, d = ri.pop(i)
        det = a * d - b * c
        ia, ib, ic, id_ = d / det, -b / det, -c / det, a / det
        y0, y1 = rhs[i]
        y0, y1 = ia * y0 + ib * y1, ic * y0 + id_ * y1
        # the row scaled by the inverse of its diagonal block
        for j, (p, q, r, s) in ri.items():
            ri[j] = (ia * p + ib * r, ia * q + ib * s, ic * p + id_ * r, ic * q + id_ * s)
        rhs[i] = (y0, y1)
        items = list(ri.items())
        for k, _ in items:
            rk = rows[k]
            a, b, c, d = rk.pop(i)
            z0, z1 = rhs[k]
            rhs[k] = (z0 - a * y0 - b * y1, z1 - c * y0 - d * y1)
            for j, (p, q, r, s) in items:
                e, f, g, h = rk.get(j, (0.0, 0.0, 0.0, 0.0))
                rk[j] = (e - a * p - b * r, f - a * q - b * s, g - c * p - d * r, h - c * q - d * s)
    x = {}
    rest = sorted(left)
    if rest:
        at = {i: k for k, i in enumerate(rest)}
        M, v = np.zeros((2 * len(rest), 2 * len(rest))), np.zeros(2 * len(rest))
        for i in rest:
            k = 2 * at[i]
            v[k:k + 2] = rhs[i]
            for j, blk in rows[i].items():
                M[k:k + 2, 2 * at[j]:2 * at[j] + 2] = np.reshape(blk, (2, 2))
        s = np.linalg.solve(M, v)
        x = {i: (s[2 * k], s[2 * k + 1]) for i, k in at.items()}
    for i in reversed(done):
        y0, y1 = rhs[i]
        for j, (p, q, r, s) in rows[i].items():
            x0, x1 = x[j]
            y0 -= p * x0 + q * x1
            y1 -= r * x0 + s * x1
        x[i] = (y0, y1)
    return x


def _root(g):
    polar = hasattr(g, "bus_type")
    kind = g.bus_type if polar else g.node_type
    n, col = g.n, g.col
    row = np.repeat(np.arange(n), np.diff(g.row_ptr))
    m = np.where(kind == pfgen.PQ, 1.0, g.v_mag)
    V = m * np.exp(1j * (np.where(kind == pfgen.SLACK, g.v_ang, 0.0) if polar else g.v_ang))
    free = kind != pfgen.SLACK
    nodes = np.flatnonzero(free).tolist()
    keep = free[row] & free[col]
    diag = row == col

    def complex_sum(w):
        return np.bincount(row, w.real, n) + 1j * np.bincount(row, w.imag, n)

    last = math.inf
    for _ in range(30):
        inj = complex_sum(g.y * V[col])
        mag = np.abs(V)
        if polar:
            S, dS = g.p_sp + 1j * g.q_sp, np.zeros(n, complex)
        else:
            zc = g.zip[:, :3] + 1j * g.zip[:, 3:]
            S = -(zc[:, 0] * mag ** 2 + zc[:, 1] * mag + zc[:, 2])
            dS = -(2 * zc[:, 0] + zc[:, 1] / mag)  # dS/d|V| over |V|, times Re V or Im V below
        F = S - V * np.conj(inj)
        # d(V conj(I))/d(Re V_j), d(Im V_j): V_i conj(Y_ij) (1, -j), plus conj(I_i) (1, j) on the diagonal
        t = V[row] * np.conj(g.y)
        de, df = t.copy(), -1j * t
        de[diag] += np.conj(inj) - dS * V.real
        df[diag] += 1j * np.conj(inj) - dS * V.imag
        J = np.stack([de.real, df.real, de.imag, df.imag], 1)
        f = np.stack([F.real, F.imag], 1)
        pv = kind == pfgen.PV
        J[pv[row], 2:] = 0.0
        J[diag & pv[row], 2:] = np.stack([2 * V.real, 2 * V.imag], 1)[pv]
        f[pv, 1] = (m ** 2 - mag ** 2)[pv]
        rows = {i: {} for i in nodes}
        for i, j, blk in zip(row[keep].tolist(), col[keep].tolist(), map(tuple, J[keep].tolist())):
            rows[i][j] = blk
        rhs = {i: tuple(v) for i, v in zip(nodes, f[free].tolist())}
        x = _solve_blocks(nodes, rows, rhs)
        dV = np.array([complex(*x[i]) for i in nodes])
        V[nodes] += dV
        step = float(np.max(np.abs(dV)))
        if step < 1e-13 or (step < 1e-9 and step > 0.1 * last):
            return V
        last = step
    raise RuntimeError("no root found from the flat start")


# buses of the largest grid, and of all grids of a mix, whose root is formed
# here (about 20 s of host time)
ROOT_BUSES = 25000


def exact(case, seed):
    if case["count"] > 60:
        return None
    grids = _inputs(case, seed)
    V, left = [], ROOT_BUSES
    for k in np.argsort([g.n for g in grids], kind="stable"):
        ok = grids[k].n <= left
        left -= grids[k].n if ok else 0
        V.append((k, _root(grids[k]) if ok else None))
    if all(v is None for _, v in V):
        return None
    return {"status": np.zeros(len(grids), np.int32), "V": [v for _, v in sorted(V, key=lambda p: p[0])]}
