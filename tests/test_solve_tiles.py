"""The one-launch solve on patterns and arguments beside the usual ones: a solution that is written over
its right-hand side (b is copied first where an entry of it could be overwritten before it is
read), systems side by side, a right-hand side with infinities or with the bits of the exchange
vectors' "not written" mark, a long chain, lists beyond the positions.  And the schedules of the
budgets that the library uses, replayed on the CPU, and on the GPU against the solve without
tiles."""
import os
import pathlib
import shutil
import subprocess

import numpy as np
import pytest

import kkt_synth as ks
import oracle
import paper_2401_13926_amd as P

ROOT = pathlib.Path(__file__).resolve().parents[1]
CSRC = ROOT / "paper_2401_13926_amd" / "csrc"
REF_LDS = 32_512  # LDS bytes of a refactorization tile
# LDS bytes of a solve tile and of one with its dense range: below 250,000 rows, and from there
SOL_LDS = {"small": (12_288, 20_000), "large": (16_384, 26_000)}


def compiled(tmp_path_factory, name):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    out = tmp_path_factory.mktemp("tiles") / name
    cmd = [gxx, "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
           "-ffp-contract=off", "-I", str(CSRC), "-o", str(out), str(ROOT / "tests" / "sanitize" / (name + ".cpp")),
           str(CSRC / "analysis.cpp")]
    subprocess.run(cmd, check=True)
    return out


@pytest.fixture(scope="module")
def order_driver(tmp_path_factory):
    return compiled(tmp_path_factory, "solve_order_driver")


@pytest.fixture(scope="module")
def replay_driver(tmp_path_factory):
    return compiled(tmp_path_factory, "solve_tiles_driver")


def cycles(n, k=7, c=2.0):
    """n / k blocks that are cyclic permutations: every pivot off the diagonal, every row a tree of its
    own (k = 2: symmetric)."""
    i = np.arange(n)
    v = np.full(n, c) * (1.0 + 0.25 * (i // k % 3))
    return np.arange(n + 1, dtype=np.int64), (i // k * k + (i % k + 1) % k).astype(np.int64), v


def stacked(p, k):
    """k copies of the system of p side by side."""
    rp = np.concatenate([[0]] + [p.rowptr[1:] + c * p.rowptr[-1] for c in range(k)]).astype(np.int64)
    return rp, np.concatenate([p.colidx + c * p.N for c in range(k)]), np.tile(p.system(1)[0], k)


def paths(n, k):
    """n / k paths of k vertices."""
    i = np.arange(n - 1)
    i = i[(i + 1) % k != 0]
    rows, cols = np.concatenate([np.arange(n), i, i + 1]), np.concatenate([np.arange(n), i + 1, i])
    vals = np.concatenate([np.full(n, 4.0), np.full(2 * len(i), -1.0)])
    order = np.lexsort((cols, rows))
    return np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))]).astype(np.int64), cols[order], vals[order]


def twisted(n, k):
    """Paths of k vertices with the rows of each moved on by k / 2: off-diagonal pivots (K has a zero diagonal), and fill."""
    rp, ci, v = paths(n, k)
    i = np.arange(n)
    src = i // k * k + (i % k + k // 2) % k
    rows = [np.arange(rp[r], rp[r + 1]) for r in src]
    take = np.concatenate(rows)
    return np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64), ci[take], v[take]


# systems side by side: (system, size of one)
FORESTS = {
    "kkt-100": lambda: (stacked(ks.small_kkt(60, 40, 7), 100), 100),
    "kkt-1000": lambda: (stacked(ks.small_kkt(600, 400, 7), 6), 1000),
    "path-500": lambda: (paths(10_000, 500), 500),
    "path-50": lambda: (paths(10_000, 50), 50),
}


def system(case, n=7_000):
    if case in FORESTS:
        return FORESTS[case]()[0]
    if case == "path":
        return paths(n, n)
    if case == "twisted":
        return twisted(n // 9 * 9, 9)
    if case == "cycles":
        return cycles(n // 7 * 7)
    if case == "pairs":
        return cycles(n, 2)
    p = ks.small_kkt(1801, 1203, 9)
    return p.rowptr, p.colidx, p.system(1)[0]


def look(order_driver, tmp_path, case, sol, *more):
    rp, ci, v = system(case)
    f = tmp_path / "in.bin"
    with open(f, "wb") as fh:
        fh.write(np.array([len(rp) - 1, len(ci)], np.int64).tobytes() + np.array([1e-10], np.float64).tobytes())
        fh.write(np.array([0, REF_LDS], np.int32).tobytes() + np.array(SOL_LDS[sol], np.int64).tobytes())
        fh.write(rp.astype(np.int64).tobytes() + ci.astype(np.int32).tobytes() + v.tobytes())
    r = subprocess.run([str(order_driver), str(f), *map(str, more)], capture_output=True, text=True, env=dict(os.environ), timeout=600)
    assert r.returncode == 0, r.stderr[-4000:]
    return {k: int(x) for k, x in (kv.split("=") for kv in r.stdout.split())}


@pytest.mark.parametrize("sol", sorted(SOL_LDS))
@pytest.mark.parametrize("case", ["cycles", "twisted", "kkt"])
def test_overwriting_is_seen(order_driver, tmp_path, case, sol):
    out = look(order_driver, tmp_path, case, sol)
    assert out["tiles"] > 1
    assert (out["offdiag"] > 0) == (case != "kkt"), out
    assert (out["early"] > 0) == (case == "cycles") or case == "twisted", out  # (its trees may fill whole tiles)
    assert out["same"] == (out["offdiag"] > 0) and out["shifted"] == 1 and out["apart"] == 0, out


@pytest.mark.parametrize("sol", sorted(SOL_LDS))
@pytest.mark.parametrize("case", ["kkt", "path"] + sorted(FORESTS))
def test_dense_ranges_keep_to_one_tree(order_driver, tmp_path, case, sol):
    out = look(order_driver, tmp_path, case, sol)
    assert out["tiles"] > 0 and out["mixed"] == 0, out
    assert case in FORESTS or out["dense"] > 0, out


REPLAYED = ["kkt", "path", "twisted"] + sorted(FORESTS)
# the library's budgets, and one of a few rows a tile: many layers of the solve, mostly externals
BUDGETS = dict(SOL_LDS, tiny=(1_200, 2_400))


@pytest.mark.parametrize("sol", sorted(BUDGETS))
@pytest.mark.parametrize("case", REPLAYED)
def test_replay_of_the_solve_tiles(replay_driver, tmp_path, case, sol):
    rp, ci, v1 = system(case, 3_500)
    v2 = v1 * (1.0 + 0.01 * np.random.default_rng(2).standard_normal(len(v1)))
    f = tmp_path / "in.bin"
    with open(f, "wb") as fh:
        fh.write(np.array([len(rp) - 1, len(ci)], np.int64).tobytes() + np.array([1e-10], np.float64).tobytes())
        fh.write(np.array([0, REF_LDS], np.int32).tobytes() + rp.astype(np.int64).tobytes())
        fh.write(ci.astype(np.int32).tobytes() + v1.tobytes() + v2.tobytes())
    r = subprocess.run([str(replay_driver), str(f), str(tmp_path / "factors.bin")], capture_output=True, text=True,
                       env=dict(os.environ, SOL_LDS=str(BUDGETS[sol][0]), SOL_DENSE_LDS=str(BUDGETS[sol][1])), timeout=600)
    assert r.returncode == 0, r.stderr[-4000:]
    out = dict(kv.split("=", 1) for kv in r.stdout.split())
    assert int(out["tiles"]) > 0 and out["refactor"] == "ok", out
    fac = np.fromfile(tmp_path / "factors.bin", np.float64)
    lx, ux, _ = oracle.LU(rp, ci, v1).refactor64(rp, ci, v2)
    assert np.array_equal(fac[:lx.size], lx) and np.array_equal(fac[lx.size:], ux)
    # sums in another order than plain substitution's, along chains of up to a few hundred rows
    assert out["solve"].startswith("ok:") and float(out["solve"][3:]) <= 1e-9, out["solve"]


def test_no_tiles_beyond_the_positions(order_driver, tmp_path):
    """Lists longer than a position can name (2^31 in earnest): no tiles, as for a node that does not fit."""
    longest = look(order_driver, tmp_path, "kkt", "small")["longest"]
    assert look(order_driver, tmp_path, "kkt", "small", longest)["tiles"] > 0
    assert look(order_driver, tmp_path, "kkt", "small", longest - 1)["tiles"] == 0


def test_analysis_of_a_long_chain():
    """An elimination tree that is one path (thousands of layers of tiles): the tiles cost a part of what
    the analysis costs without them, not a pass over the tree per layer."""
    rp, ci, v = paths(600_000, 600_000)

    def seconds(**opts):
        return min(P.Solver(rp, ci, v, **opts).info()["analysis_seconds"] for _ in range(2))

    with_tiles, without = seconds(), seconds(tile_lds_kib=32)
    # 1.1 times as long; 4.4 times with passes over all nodes for each layer
    assert with_tiles < 2.5 * without, (with_tiles, without)


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [P.PREC_FP64, P.PREC_MIXED])
@pytest.mark.parametrize("case", ["cycles", "pairs", "twisted", "kkt"])
def test_direct_solve_over_its_right_hand_side(case, precision):
    """x in b's place, and one entry after it, against x in an array of its own: the same bits."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("in place", case, precision, flush=True)
    rp, ci, v = system(case, 200_000)
    n = len(rp) - 1
    s = P.Solver(rp, ci, v, precision=precision).bind("cuda")
    s.refactor(torch.as_tensor(v, device="cuda"))
    b = torch.as_tensor(np.random.default_rng(3).standard_normal(n), device="cuda")
    want = s.direct_solve(b)
    assert torch.isfinite(want).all()
    for solve in (s.direct_solve, s.direct_solve_noalloc):
        for shift in (0, 1):
            for _ in range(3):
                buf = torch.empty(n + 1, dtype=torch.float64, device="cuda")
                buf[:n] = b
                solve(buf[:n], buf[shift:shift + n])
                assert torch.equal(buf[shift:shift + n], want)


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [P.PREC_FP64, P.PREC_MIXED])
@pytest.mark.parametrize("case", REPLAYED + ["cycles", "pairs"])
def test_solve_with_tiles_against_without(case, precision):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("tiles against none", case, precision, flush=True)
    rp, ci, v = system(case, 14_000)
    b = torch.as_tensor(np.random.default_rng(3).standard_normal(len(rp) - 1), device="cuda")
    x = []
    for lds in (0, 32):  # 0: tiles
        s = P.Solver(rp, ci, v, precision=precision, tile_lds_kib=lds).bind("cuda")
        s.refactor(torch.as_tensor(v, device="cuda"))
        x.append(s.direct_solve(b))
    # the replay's bound, at the factors' unit roundoff for FP32 (2^29 times as large; the KKT systems
    # lose all digits there)
    if precision == P.PREC_FP64:
        assert float((x[0] - x[1]).abs().max()) <= 1e-9 * float(x[1].abs().max())
    elif "kkt" not in case:
        assert float((x[0] - x[1]).abs().max()) <= 1e-4 * float(x[1].abs().max())
    assert bool(torch.isfinite(x[0]).all())


SENTINEL = np.array([0x7FF4DEADBEEF0001], np.uint64).view(np.float64)[0]


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [P.PREC_FP64, P.PREC_MIXED])
@pytest.mark.parametrize("where", ["one", "all"])
def test_right_hand_side_with_the_unwritten_mark(where, precision):
    """A NaN like any other: the direct solve passes it on, the solve refuses b, the handle goes on."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("sentinel in b", where, precision, flush=True)
    # a NaN in one of 30 systems side by side leaves the others finite
    p, k = ks.small_kkt(60, 40, 7), 30
    rp, ci, v = stacked(p, k)
    s = P.Solver(rp, ci, v, precision=precision).bind("cuda")
    s.refactor(torch.as_tensor(v, device="cuda"))
    b0 = np.random.default_rng(3).standard_normal(k * p.N)

    def on_gpu(b):
        return torch.as_tensor(b.view(np.int64), device="cuda").view(torch.float64)

    want = s.direct_solve(on_gpu(b0)).cpu().numpy()
    assert np.isfinite(want).all()
    rows = range(p.N * 4, p.N * 5) if where == "one" else [None]  # every row of a system in turn: leaves, roots
    for row in rows:
        mark, nan = b0.copy(), b0.copy()
        mark[slice(None) if row is None else row] = SENTINEL
        nan[slice(None) if row is None else row] = np.nan
        assert (mark.view(np.int64) != b0.view(np.int64)).any()
        ref = s.direct_solve(on_gpu(nan)).cpu().numpy()
        assert np.isnan(ref).any()
        x = on_gpu(np.zeros_like(b0))
        for got in (s.direct_solve(on_gpu(mark)), s.direct_solve_noalloc(on_gpu(mark), x)):
            got = got.cpu().numpy()
            assert np.array_equal(np.isnan(got), np.isnan(ref))
            assert np.array_equal(got[~np.isnan(ref)], want[~np.isnan(ref)])
    with pytest.raises(P.KKTError) as e:
        s.solve(on_gpu(mark))
    assert e.value.args and "non-finite" in str(e.value)
    x, info = s.solve(on_gpu(b0))
    assert info["converged"] == 1 and bool(torch.isfinite(x).all())


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [P.PREC_FP64, P.PREC_MIXED])
@pytest.mark.parametrize("case", sorted(FORESTS))
def test_infinity_stays_in_its_system(case, precision):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("infinity in b", case, precision, flush=True)
    (rp, ci, v), size = FORESTS[case]()
    n = len(rp) - 1
    s = P.Solver(rp, ci, v, precision=precision).bind("cuda")
    s.refactor(torch.as_tensor(v, device="cuda"))
    rng = np.random.default_rng(5)
    b0 = rng.standard_normal(n)
    want = s.direct_solve(torch.as_tensor(b0, device="cuda")).cpu().numpy()
    for i in rng.integers(0, n, 12):
        b = b0.copy()
        b[i] = np.inf
        got = s.direct_solve(torch.as_tensor(b, device="cuda")).cpu().numpy()
        other = np.arange(n) // size != i // size
        assert np.array_equal(got[other], want[other])
