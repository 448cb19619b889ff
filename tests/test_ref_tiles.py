"""The tile schedules of the refactorization and of the solves: replayed on the CPU (a driver built with
AddressSanitizer and UndefinedBehaviorSanitizer) it gives the oracle's static-pivot
refactorization bit for bit, over tile budgets from one that holds a handful of nodes (many
layers, mostly externals) to one that holds the whole system, and both sweeps give plain
substitution's solution; patterns it does not serve keep the
hand-out items.  On the GPU the tile kernel's factors equal the oracle's and the hand-out
kernel's."""
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


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    out = tmp_path_factory.mktemp("tiles") / "ref_tiles_driver"
    cmd = [gxx, "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
           "-ffp-contract=off", "-I", str(CSRC), "-o", str(out),
           str(ROOT / "tests" / "sanitize" / "ref_tiles_driver.cpp"), str(CSRC / "analysis.cpp")]
    subprocess.run(cmd, check=True)
    return out


def run(driver, tmp_path, p, v1, v2, lds, tau=1e-10, ordering=0):
    f = tmp_path / "in.bin"
    with open(f, "wb") as fh:
        fh.write(np.array([p.N, p.colidx.size], np.int64).tobytes() + np.array([tau], np.float64).tobytes())
        fh.write(np.array([ordering, lds], np.int32).tobytes())
        fh.write(p.rowptr.astype(np.int64).tobytes() + p.colidx.astype(np.int32).tobytes())
        fh.write(v1.tobytes() + v2.tobytes())
    r = subprocess.run([str(driver), str(f), str(tmp_path / "factors.bin")], capture_output=True, text=True,
                       env=dict(os.environ), timeout=600)
    assert r.returncode == 0, r.stderr[-4000:]
    return dict(kv.split("=", 1) for kv in r.stdout.split() if "=" in kv)


CASES = {
    "1x1": lambda: ks.small_kkt(6, 1, 3),
    "tiny": lambda: ks.small_kkt(40, 21, 5),
    "3k": lambda: ks.small_kkt(1801, 1203, 9),
    "mild": lambda: ks.moderate_kkt(2000, 1500),
    "7k": lambda: ks.make_pattern(1),
}


@pytest.mark.parametrize("lds", [4_500, 32_768, 153_600])
@pytest.mark.parametrize("case", sorted(CASES))
def test_tiles_replay_matches_oracle(driver, tmp_path, case, lds):
    p = CASES[case]()
    v1, v2 = p.system(1)[0], p.system(2)[0]
    out = run(driver, tmp_path, p, v1, v2, lds)
    if lds == 4_500 and int(out["tiles"]) == 0:
        return  # one node of the larger cases does not fit so small a tile: the items serve it
    assert int(out["tiles"]) > 0 and out["refactor"] == "ok", out
    fac = np.fromfile(tmp_path / "factors.bin", np.float64)
    lx, ux, guarded = oracle.LU(p.rowptr, p.colidx, v1).refactor64(p.rowptr, p.colidx, v2)
    assert np.array_equal(fac[:lx.size], lx) and np.array_equal(fac[lx.size:], ux)
    assert int(out["guarded"]) == guarded
    # sums in another order than plain substitution's: rounding of a few dozen terms a row, along
    # chains of about a hundred rows
    assert out["solve"].startswith("ok:") and float(out["solve"][3:]) <= 1e-9, out["solve"]


def test_tiles_replay_guards_as_the_oracle(driver, tmp_path):
    # system 2 with D = 0 and J = 0 in places: pivots that vanish or fall under the guard
    p = ks.small_kkt(900, 600, 13)
    v1, v2 = p.system(1)[0], p.system(2)[0].copy()
    row = np.repeat(np.arange(p.N), np.diff(p.rowptr))
    dead = (row % 7 == 3) & (row == p.colidx)
    v2[dead] = 0.0
    v2[(row % 11 == 5) | (p.colidx % 11 == 5)] *= 1e-30
    out = run(driver, tmp_path, p, v1, v2, 32_768)
    assert out["refactor"] == "ok"
    lx, ux, guarded = oracle.LU(p.rowptr, p.colidx, v1).refactor64(p.rowptr, p.colidx, v2)
    fac = np.fromfile(tmp_path / "factors.bin", np.float64)
    assert guarded > 0 and int(out["guarded"]) == guarded
    assert np.array_equal(fac[:lx.size], lx) and np.array_equal(fac[lx.size:], ux)


def test_patterns_without_tiles(driver, tmp_path):
    # off-diagonal pivots (L and U patterns differ), and a column too long for a tile
    p = ks.small_kkt(900, 600, 13)
    assert int(run(driver, tmp_path, p, p.system(1)[0], p.system(2)[0], 32_768, tau=0.1)["tiles"]) == 0
    a = ks.ArrowKKT(4000, 1500, 2500, seed=1)
    assert int(run(driver, tmp_path, a, a.system(1)[0], a.system(2)[0], 32_768)["tiles"]) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [P.PREC_FP64, P.PREC_MIXED])
@pytest.mark.parametrize("case", ["tiny", "3k", "mild", "7k", "guarded"])
def test_tile_kernel_matches_items_and_oracle(case, precision):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("tile kernel", case, precision, flush=True)
    p = ks.small_kkt(900, 600, 13) if case == "guarded" else CASES[case]()
    v1, v2 = p.system(1)[0], p.system(2)[0].copy()
    if case == "guarded":
        row = np.repeat(np.arange(p.N), np.diff(p.rowptr))
        v2[(row % 7 == 3) & (row == p.colidx)] = 0.0
    f = oracle.LU(p.rowptr, p.colidx, v1)
    olx, oux, guarded = (f.refactor32 if precision else f.refactor64)(p.rowptr, p.colidx, v2)
    got = []
    for narrow in (0, 1):  # 0: tiles; 1: the hand-out of single columns
        s = P.Solver(p.rowptr, p.colidx, v1, precision=precision, narrow_columns=narrow).bind("cuda")
        for _ in range(2):
            s.refactor(torch.as_tensor(v1, device="cuda"))
            s.refactor(torch.as_tensor(v2, device="cuda"))
        torch.cuda.synchronize()
        got.append(s.factor_values(1 if precision else 0))
    for lx, ux in got:
        assert np.array_equal(lx, olx.astype(np.float64)) and np.array_equal(ux, oux.astype(np.float64))
    if case == "guarded" and not precision:
        assert guarded > 0
