"""Standalone products on both sides of the length of x at which a tile's entries are
streamed (5/4 of an XCD's L2 of 4 MB: 655 360 values in FP64, 1 310 720 in FP32), and
the single-QP kernels on both sides of theirs (8 n bytes of 3/2 L2: n = 786 432).

A row has at most 8 entries of size about 1: 8 eps of the largest |y| in FP64; with
FP32 values and x, 2 * 2^-24 of each of the 8 products and no more than 8 of them per
row: 1e-6 of the largest |y|.  Solves: five iterations, sums of at most n terms in
another order than the oracle's, 1e-10.
"""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2405_16160_amd import instances as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2405_16160_amd import pdhcg  # noqa: E402


def banded(nrows, ncols, rng, per_row):
    """rows of 0 to per_row entries in random columns"""
    lens = rng.integers(0, per_row + 1, nrows)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    col = rng.integers(0, ncols, int(rp[-1])).astype(np.int64)
    row = np.repeat(np.arange(nrows), lens)
    key = np.unique(row * np.int64(ncols) + col)   # (sorted, without repeats in a row)
    row, col = key // ncols, key % ncols
    rp = np.concatenate([[0], np.cumsum(np.bincount(row, minlength=nrows))]).astype(np.int64)
    return I.CSR(nrows, ncols, rp, col.astype(np.int32), rng.standard_normal(len(key)))


def diagonal(n, rng):
    return I.CSR(n, n, np.arange(n + 1, dtype=np.int64), np.arange(n, dtype=np.int32), 1.0 + rng.random(n))


@pytest.mark.parametrize("n", [655_360, 655_361, 1_310_720, 1_310_721])
def test_product_at_the_line(n):
    rng = np.random.default_rng(n)
    m = 300_001
    qp = I.QP(diagonal(n, rng), banded(m, n, rng, 8), np.ones(m), np.ones(n))
    print(f"[spmv line] n={n}", flush=True)
    h = pdhcg.Solver(qp, pdhcg.Settings(precision=1))
    x = rng.standard_normal(n)
    for which, want in ((0, qp.Q.val * x), (1, O.matvec(qp.A, x))):
        for precision, tol in ((0, 8 * 2.3e-16), (1, 1e-6)):
            y = h.spmv(which, torch.tensor(x, device="cuda"), precision=precision).cpu().numpy()
            assert np.abs(y - want).max() <= tol * np.abs(want).max()
    h.close()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n", [786_432, 786_433])
def test_solve_at_the_line(n, precision):
    rng = np.random.default_rng(n)
    m = 200_003
    qp = I.QP(diagonal(n, rng), banded(m, n, rng, 8), np.ones(m), rng.standard_normal(n))
    print(f"[solve line] n={n} precision={precision}", flush=True)
    h = pdhcg.Solver(qp, pdhcg.Settings(tol_rel_kkt=1e-14, max_iters=5, precision=precision, cg_rule=1, max_cg_iters=3))
    assert h.plan_info()["threads"] == 256
    x, y, r = h.solve()
    h.close()
    o = O.solve(qp, O.Settings(tol=1e-14, max_iters=5, cg_rule=1, max_cg=3))
    assert r["iters"] == o.iters == 5
    tol = 2e-5 if precision else 1e-10
    assert np.linalg.norm(x.cpu().numpy() - o.x) <= tol * np.linalg.norm(o.x)
    assert np.linalg.norm(y.cpu().numpy() - o.y) <= tol * max(np.linalg.norm(o.y), np.linalg.norm(o.x))
