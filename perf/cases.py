"""Performance cases of the solver library: what its users have it do, through the Python
entry points (Solver, refactor_batch, Server, HyKKT), from 1,000 to 2,000,000 unknowns.

A case is a dict of plain values:

* ``kind``: the call or calls of one pass,
    - ``step``      one system of a sequence: refactor(values), then solve(b) with refinement;
    - ``factor``    refactor(values), then one direct_solve(b) (no refinement);
    - ``direct``    direct_solve(b) alone, with factors already there (one preconditioner use);
    - ``residual``  residual(b, x) of a refactored system;
    - ``batch``     refactor_batch of ``count`` systems of one pattern through a graph, then a
                    solve of each;
    - ``serve``     ``count`` requests, round robin over patterns of ``n`` + ``m`` and ``n2`` +
                    ``m2`` unknowns, submitted to a Server at once and waited for;
    - ``hykkt``     HyKKT refactor(values) and solve(b) (zero (2,2) block);
* ``n``, ``m``: primal and dual unknowns (N = n + m), ``dlog``: the barrier term D is
  log-uniform over 10^[-dlog, dlog], ``delta``: the (2,2) block is -delta I;
* ``restart``, ``precision``, ``residual``, ``gram_schmidt``: options of the solver.

The pattern and the host analysis of its first system are what a user's program makes once;
a state holds a bound handle, the values of a later system and its right-hand side.
"""
from __future__ import annotations

import functools
import heapq

import numpy as np
import torch

import kkt_synth as ks
import paper_2401_13926_amd as P

#: Generator configuration of the patterns drawn here (its random streams).
CONFIG = 8


def listed():
    wide, mid, small, mild = 12.0, 10.0, 8.0, 2.0
    return [
        # one right-hand side on a tiny system: launch and dependency latency alone
        case("direct", 600, 400, small, name="direct-1k"),
        # interior-point steps of the sequence benchmarks, smallest to largest (the last one is
        # the default workload of bench.py)
        case("step", 4_000, 3_000, small, name="step-7k"),
        case("step", 35_000, 25_000, mid, name="step-60k"),
        case("step", 290_000, 210_000, wide, name="step-500k", restart=30),
        case("step", 1_150_000, 850_000, wide, name="step-2m", restart=50),
        # static refactorization with its direct solution only, at a ragged serving size
        case("factor", 85_757, 62_100, mid, name="factor-148k"),
        # the factors used as a preconditioner for another right-hand side
        case("direct", 290_000, 210_000, wide, name="direct-500k", restart=30),
        # a user's own accuracy check, in double-double
        case("residual", 126_606, 91_680, mid, name="residual-dd-218k", residual="dd"),
        # optimizer instances of one pattern, refactored together
        case("batch", 44_909, 32_520, mid, name="batch-4x77k", count=4),
        # FP32 factors as the preconditioner, on the family where they suffice
        case("step", 35_000, 25_000, mild, name="mixed-60k", delta=1.0, precision="mixed"),
        # the second solver: CG on the Schur complement
        case("hykkt", 35_000, 25_000, mild, name="hykkt-60k", delta=0.0),
        # a burst of requests on two patterns
        case("serve", 4_060, 2_940, mid, name="serve-16", count=16, n2=44_909, m2=32_520),
    ]


def case(kind, n, m, dlog, delta=ks.DUAL_REG, restart=10, **more):
    c = {"kind": kind, "n": n, "m": m, "dlog": dlog, "delta": delta, "restart": restart, "precision": "fp64",
         "residual": "fp64", "gram_schmidt": "cgs2"}
    c.update(more)
    return c


def draw(rng):
    """A case of the listed kinds: N log-uniform (1,000 to 1,000,000 where one system is
    handled), any remainder, D as wide as the sequences of that size have it."""

    def size(lo, hi):
        N = int(round(lo * (hi / lo) ** rng.random()))
        n = int(round(rng.uniform(0.55, 0.62) * N))
        return n, N - n

    def width(N):
        return 8.0 if N < 20_000 else 10.0 if N < 250_000 else 12.0

    kind = rng.choice(["step", "step", "step", "factor", "direct", "direct", "residual", "batch", "mixed", "hykkt"])
    if kind == "batch":
        n, m = size(5_000, 150_000)
        return case("batch", n, m, width(n + m), count=rng.randint(2, 8))
    if kind == "hykkt":
        n, m = size(5_000, 150_000)
        return case("hykkt", n, m, 2.0, delta=0.0)
    n, m = size(1_000, 1_000_000)
    restart = 10 if n + m < 250_000 else 30
    if kind == "mixed":
        return case("step", n, m, 2.0, delta=1.0, restart=restart, precision="mixed")
    if kind == "step":
        return case("step", n, m, width(n + m), restart=restart, residual=rng.choice(["fp64", "fp64", "dd"]),
                    gram_schmidt=rng.choice(["cgs2", "cgs2", "dcgs2"]))
    if kind == "residual":
        return case("residual", n, m, width(n + m), restart=restart, residual=rng.choice(["fp64", "dd"]))
    return case(kind, n, m, width(n + m), restart=restart)


# --- what a user's program has before the call -------------------------------------------


def _pattern(n, m, c):
    return ks.make_pattern(CONFIG, 0, n=n, m=m, dlog=(-c["dlog"], c["dlog"]), delta=c["delta"])


def _options(c):
    return dict(restart=c["restart"], precision=P.PREC_MIXED if c["precision"] == "mixed" else P.PREC_FP64,
                residual=P.RESID_DD if c["residual"] == "dd" else P.RESID_FP64,
                gram_schmidt=P.GS_DCGS2 if c["gram_schmidt"] == "dcgs2" else P.GS_CGS2)


@functools.lru_cache(maxsize=12)
def _analysed(n, m, dlog, delta, options):
    """The analysed handle of a pattern; states bind clones of it."""
    p = _pattern(n, m, {"dlog": dlog, "delta": delta})
    return P.Solver(p.rowptr, p.colidx, p.system(1)[0], **dict(options))


def _handle(c):
    base = _analysed(c["n"], c["m"], c["dlog"], c["delta"], tuple(sorted(_options(c).items())))
    return base.clone().bind("cuda")


def _systems(c, seed):
    """(pattern, values, b) of every system of a state, on the host, from the seed."""
    count = c.get("count", 1)
    out = []
    for k in range(count):
        n, m = (c["n2"], c["m2"]) if "n2" in c and k % 2 else (c["n"], c["m"])
        p = _pattern(n, m, c)
        # a later system of the sequence: its own D, 1 % other H and J values, its own b
        v, b = p.system(2 + (int(seed) * 16 + k) % 2_000_000_000)
        out.append((p, v, b))
    return out


def _near_solution(p, v, seed):
    """(b, x) with b = K x0 for a drawn x0 and x = x0 up to relative 1e-8: what a residual is
    taken of when a solution is looked at."""
    rng = np.random.Generator(np.random.PCG64(np.random.SeedSequence([CONFIG, int(seed)])))
    x0 = rng.standard_normal(p.N)
    b = np.add.reduceat(v * x0[p.colidx], p.rowptr[:-1])
    return b, x0 * (1.0 + 1e-8 * rng.standard_normal(p.N))


class State:
    def __init__(self, c, seed):
        self.kind = c["kind"]
        systems = _systems(c, seed)
        self.values = [torch.as_tensor(v, device="cuda") for _, v, _ in systems]
        self.b = [torch.as_tensor(b, device="cuda") for _, _, b in systems]
        self.x = [torch.empty_like(b) for b in self.b]
        p = systems[0][0]
        if self.kind == "hykkt":
            self.solver = P.HyKKT(p.rowptr, p.colidx, p.system(1)[0], p.n).bind("cuda")
        elif self.kind == "serve":
            self.server = P.Server(8 << 30, workers=4)
            self.patterns = [self.server.add_pattern(q.rowptr, q.colidx, q.system(1)[0], **_options(c))
                             for q in (p, systems[1][0])]
        elif self.kind == "batch":
            self.solvers = [_handle(c) for _ in systems]
        else:
            self.solver = _handle(c)
            if self.kind in ("direct", "residual"):
                self.solver.refactor(self.values[0])
            if self.kind == "residual":
                b, x = _near_solution(p, systems[0][1], seed)
                self.b, self.x = [torch.as_tensor(b, device="cuda")], [torch.as_tensor(x, device="cuda")]
                self.r = torch.empty_like(self.b[0])
        torch.cuda.synchronize()


def prepare(case, seed):
    return State(case, seed)


def run(s):
    if s.kind == "direct":
        return s.solver.direct_solve(s.b[0], s.x[0])
    if s.kind == "residual":
        return s.solver.residual(s.b[0], s.x[0], s.r)
    if s.kind == "factor":
        s.solver.refactor(s.values[0])
        return s.solver.direct_solve(s.b[0], s.x[0])
    if s.kind in ("step", "hykkt"):
        s.solver.refactor(s.values[0])
        x, info = s.solver.solve(s.b[0], s.x[0], allow_noconv=True)
        return {"x": x, "converged": info["converged"]}
    if s.kind == "batch":
        P.refactor_batch(s.solvers, s.values, graph=True)
        infos = [h.solve(b, x, allow_noconv=True)[1] for h, b, x in zip(s.solvers, s.b, s.x)]
        return {"x": s.x, "converged": [i["converged"] for i in infos]}
    tickets = [s.server.submit(s.patterns[k % 2], v, b, x)
               for k, (v, b, x) in enumerate(zip(s.values, s.b, s.x))]
    done = [s.server.wait(t) for t in tickets]
    return {"x": s.x, "converged": [info["converged"] for _, info, _ in done]}


# --- what a pass cannot do without ------------------------------------------------------


def work(case):
    """Bytes and operations of one pass, each array of a stage counted once: K's values into
    the factors, the factors once per sweep pair, K once per product or residual.  These
    patterns have 6.1 factor entries and 7 multiply-subtract updates per unknown under minimum
    degree, and a step takes two refinement iterations (none in the mild family, three with
    FP32 factors there; about 200 CG iterations for HyKKT)."""
    kind, total_b, total_f = case["kind"], 0.0, 0.0
    for k in range(case.get("count", 1)):
        n, m = (case["n2"], case["m2"]) if "n2" in case and k % 2 else (case["n"], case["m"])
        N = n + m
        nnz = 2 * round(1.5 * n) + n + 7 * m
        f, word = 6.1 * N, 4 if case["precision"] == "mixed" else 8
        factor = (8 * nnz + word * f, 2 * 7 * N + f)
        pair = ((word + 4) * f + 16 * N, 2 * f)
        product = (12 * nnz + 24 * N, 2 * nnz)
        if kind == "hykkt":
            # H_gamma (n rows, about 9 entries a row, 25 in its factors) and J products
            f = 25.0 * n
            parts = [(8 * nnz + 8 * f, 2 * 150 * n + f)]
            parts += 202 * [(12 * f + 16 * n, 2 * f), (2 * 36 * m + 16 * n + 80 * m, 16 * m)]
        elif kind == "residual":
            parts = [product]
        elif kind == "direct":
            parts = [pair]
        elif kind == "factor":
            parts = [factor, pair]
        else:
            it = 3 if case["precision"] == "mixed" else 2
            parts = [factor] + (1 + it) * [pair] + (2 + it) * [product]
        total_b += sum(p[0] for p in parts)
        total_f += sum(p[1] for p in parts)
    return {"bytes": total_b, "flops": total_f}


# --- the same in 64 bits, without the library -------------------------------------------


def _residual(p, v, b, x):
    """b - K x, summed in extended precision."""
    terms = v.astype(np.longdouble) * np.asarray(x, np.longdouble)[p.colidx]
    return b.astype(np.longdouble) - np.add.reduceat(terms, p.rowptr[:-1])


def _exact_solution(p, v, b):
    """K^-1 b by a plain sparse L D L^T (a minimum degree order, diagonal pivots: K is
    quasi-definite) and refinement with extended-precision residuals until it stands still."""
    N = p.N
    rp, ci = p.rowptr.tolist(), p.colidx.tolist()
    vv = v.tolist()
    rows = [dict(zip(ci[rp[i]:rp[i + 1]], vv[rp[i]:rp[i + 1]])) for i in range(N)]
    diag = [r.pop(i, 0.0) for i, r in enumerate(rows)]
    heap = [(len(r), i) for i, r in enumerate(rows)]
    heapq.heapify(heap)
    done = [False] * N
    cols = []
    while heap:
        deg, k = heapq.heappop(heap)
        if done[k] or deg != len(rows[k]):
            continue
        done[k] = True
        near = rows[k]
        cols.append((k, list(near.items())))
        d = diag[k]
        ids = list(near)
        for a, i in enumerate(ids):
            ri = rows[i]
            del ri[k]
            l = near[i] / d
            diag[i] -= l * near[i]
            for j in ids[a + 1:]:
                t = ri.get(j, 0.0) - l * near[j]
                ri[j] = t
                rows[j][i] = t
        for i in ids:
            heapq.heappush(heap, (len(rows[i]), i))

    def apply(r):
        y = r.tolist()
        for k, items in cols:
            t = y[k] / diag[k]
            if t:
                for i, a in items:
                    y[i] -= a * t
        for k, items in reversed(cols):
            s = y[k]
            for i, a in items:
                s -= a * y[i]
            y[k] = s / diag[k]
        return np.asarray(y)

    x = np.zeros(N, np.longdouble)
    last = np.inf
    for _ in range(20):
        d = apply(_residual(p, v, b, x).astype(np.float64))
        x = x + d
        now = float(np.linalg.norm(d))
        if now <= 1e-18 * float(np.linalg.norm(x.astype(np.float64))) or now > 0.5 * last:
            break
        last = now
    return x.astype(np.float64)


def exact(case, seed):
    if case["kind"] == "residual":
        p, v, _ = _systems(case, seed)[0]
        b, x = _near_solution(p, v, seed)
        return _residual(p, v, b, x).astype(np.float64)
    if case["kind"] in ("serve", "hykkt") or (case["n"] + case["m"]) * case.get("count", 1) > 100_000:
        return None
    xs = [_exact_solution(p, v, b) for p, v, b in _systems(case, seed)]
    if case["kind"] in ("direct", "factor"):
        return xs[0]
    if case["kind"] == "step":
        return {"x": xs[0], "converged": None}
    return {"x": xs, "converged": None}
