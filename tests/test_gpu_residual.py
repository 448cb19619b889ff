"""kkt_residual on both sides of the size from which x is put into the vector order by a launch of its
own, and on rows longer than the products kept in LDS: bit-identical to the oracle's residual (same
products, same order of addition)."""
import numpy as np
import pytest

import kkt_synth as ks
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2401_13926_amd as P  # noqa: E402

LIMIT = 400_000  # rows up to which the residual kernel gathers x itself


def short_paths(n):
    """Paths of 50 vertices with random labels: (rowptr, colidx, values) of a symmetric matrix."""
    rng = np.random.default_rng(n)
    label = rng.permutation(n)
    i = np.arange(n - 1)
    i = i[(i + 1) % 50 != 0]
    off = rng.standard_normal(len(i))
    rows = np.concatenate([label, label[i], label[i + 1]])
    cols = np.concatenate([label, label[i + 1], label[i]])
    vals = np.concatenate([4.0 + rng.random(n), off, off])
    order = np.lexsort((cols, rows))
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))])
    return rowptr.astype(np.int64), cols[order].astype(np.int64), vals[order]


@pytest.mark.parametrize("resid", ["fp64", "dd"])
@pytest.mark.parametrize("case", ["arrow", LIMIT, LIMIT + 1])
def test_residual_bit_exact_around_the_gather_limit(case, resid):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("residual", case, resid, flush=True)
    dev = torch.device("cuda:0")
    if case == "arrow":  # one row of 2,500 entries and more
        a = ks.ArrowKKT(4000, 1500, 2500, seed=1)
        rp, ci, v = a.rowptr, a.colidx, a.system(1)[0]
    else:
        rp, ci, v = short_paths(case)
    n = len(rp) - 1
    s = P.Solver(rp, ci, v, residual=P.RESID_DD if resid == "dd" else P.RESID_FP64).bind(dev)
    s.refactor(torch.as_tensor(v, device=dev))
    rng = np.random.default_rng(7)
    x = rng.standard_normal(n) * 10.0 ** rng.uniform(-6, 6, n)
    b = rng.standard_normal(n)
    r = s.residual(torch.as_tensor(b, device=dev), torch.as_tensor(x, device=dev))
    torch.cuda.synchronize()
    assert np.array_equal(r.cpu().numpy(), oracle.residual(rp, ci, v, x, b, resid))
