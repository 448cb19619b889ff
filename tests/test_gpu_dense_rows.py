"""Rows of more entries than the products kept in LDS for a block of rows (2,048 for 256 rows): the
streaming kernels take such rows from memory.  ||K||_inf, the residual (bit-identical to the
oracle's: same products, same order of addition) and a refined solve, with 9 to 24 entries in
every row and with one long row among short ones, on both sides of the residual's gather limit."""
import numpy as np
import pytest

import kkt_synth as ks
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2401_13926_amd as P  # noqa: E402


def blocks(n, k):
    """n / k dense symmetric blocks of k rows, diagonally dominant."""
    rng = np.random.default_rng(k)
    nb = n // k
    a = rng.standard_normal((nb, k, k))
    a = (a + a.transpose(0, 2, 1)) / 2
    a[:, np.arange(k), np.arange(k)] += 2 * k
    cols = np.repeat(np.arange(nb * k).reshape(nb, k), k, axis=0).ravel()
    return np.arange(nb * k + 1, dtype=np.int64) * k, cols.astype(np.int64), a.ravel()


CASES = {
    "9": lambda: blocks(1_000, 9),
    "16": lambda: blocks(8_000, 16),
    "24": lambda: blocks(2_405, 24),
    "9-large": lambda: blocks(400_500, 9),
    "arrow": lambda: (lambda a: (a.rowptr, a.colidx, a.system(1)[0]))(ks.ArrowKKT(4000, 1500, 2500, seed=1)),
}


@pytest.mark.parametrize("precision", [P.PREC_FP64, P.PREC_MIXED])
@pytest.mark.parametrize("resid", ["fp64", "dd"])
@pytest.mark.parametrize("case", sorted(CASES))
def test_dense_rows(case, resid, precision):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("dense rows", case, resid, precision, flush=True)
    dev = torch.device("cuda:0")
    rp, ci, v = CASES[case]()
    n = len(rp) - 1
    s = P.Solver(rp, ci, v, precision=precision, residual=P.RESID_DD if resid == "dd" else P.RESID_FP64).bind(dev)
    s.refactor(torch.as_tensor(v, device=dev))
    rng = np.random.default_rng(7)
    x = rng.standard_normal(n) * 10.0 ** rng.uniform(-6, 6, n)
    b = rng.standard_normal(n)
    r = s.residual(torch.as_tensor(b, device=dev), torch.as_tensor(x, device=dev))
    assert np.array_equal(r.cpu().numpy(), oracle.residual(rp, ci, v, x, b, resid))
    got, info = s.solve(torch.as_tensor(b, device=dev), allow_noconv=True)
    rows = np.add.reduceat(np.abs(v), rp[:-1])  # (another order of addition: rounding of 2,500 terms at most)
    assert abs(info["knorm_inf"] - rows.max()) <= 2_500 * 2.0 ** -53 * rows.max()
    if case != "arrow":
        m = oracle.metrics(rp, ci, v, got.cpu().numpy(), b)
        assert info["converged"] == 1 and m["nrbe"] <= 1e-12, (info, m)
        assert precision == P.PREC_FP64 or info["iterations"] > 0
    bad = v.copy()
    bad[-1] = np.inf
    s.refactor(torch.as_tensor(bad, device=dev))
    with pytest.raises(P.KKTError, match="non-finite"):
        s.solve(torch.as_tensor(b, device=dev))
