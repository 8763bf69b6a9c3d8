"""Row lengths at the edges of the wave tiles of the solve kernels' sparse products.

A few iterations with a fixed number of CG steps, on few workgroups, against the
oracle's iterates.  FP64: sums of at most 3000 terms, 3000 eps = 7e-13, over 6
iterations of 3 CG steps that grow it by less than 1e2, so 1e-10; FP32 values and
gathers: 2^-24 = 6e-8 per product, so 2e-5.
"""
import numpy as np
import pytest
import scipy.sparse as sp

from oracle import oracle as O
from paper_2405_16160_amd import instances as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2405_16160_amd import pdhcg  # noqa: E402

N = 3000
LENGTHS = {
    "edges": [0, 1, 63, 64, 65, 127, 128, 129, 0, 511, 512, 513, 1023, 1024, 1025, 2, 0],
    "single": [700],
    "short": [1] * 300 + [0] * 70 + [2] * 130,
    "skewed": [3] * 200 + [400] + [3] * 200 + [2900] + [1] * 65,
    "none": [],
}


def build(name):
    rng = np.random.default_rng(11)
    lens = LENGTHS[name]
    rows = np.repeat(np.arange(len(lens)), lens)
    cols = np.concatenate([np.sort(rng.choice(N, k, replace=False)) for k in lens] + [np.zeros(0, int)]).astype(int)
    A = sp.csr_matrix((rng.standard_normal(cols.size) / np.sqrt(8.0), (rows, cols)), shape=(len(lens), N))
    # Q: a diagonal, and rows of the edge lengths (mirrored), dominated by it
    Q = sp.lil_matrix((N, N))
    for r, k in ((0, 63), (1, 512), (2, 600), (7, 1100)):
        Q[r, N - k:] = 0.5 * rng.standard_normal(k) / k
    Q = Q.tocsr()
    Q = Q + Q.T + sp.diags(1.0 + rng.random(N))
    return I.QP(I.CSR.from_scipy(I._symmetrize(Q.tocsr())), I.CSR.from_scipy(A), -rng.random(len(lens)),
                rng.standard_normal(N))


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("threads", [256, 512])
@pytest.mark.parametrize("name", list(LENGTHS))
def test_row_lengths(name, threads, precision):
    qp = build(name)
    ref = O.solve(qp, O.Settings(tol=1e-15, max_iters=6, cg_rule=1, max_cg=3))
    for form in (1, 2):
        print(f"[tiles] {name} threads={threads} precision={precision} cg_form={form}", flush=True)
        sol = pdhcg.Solver(qp, pdhcg.Settings(tol_rel_kkt=1e-15, max_iters=6, cg_rule=1, max_cg_iters=3,
                                              precision=precision, threads=threads, num_blocks=2, cg_form=form))
        x, y, r = sol.solve()
        sol.close()
        tol = 2e-5 if precision else 1e-10
        assert r["iters"] == 6
        x, y = x.cpu().numpy(), y.cpu().numpy()
        assert np.linalg.norm(x - ref.x) <= tol * np.linalg.norm(ref.x)
        assert np.linalg.norm(y - ref.y) <= tol * max(np.linalg.norm(ref.y), np.linalg.norm(ref.x))


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("lens", [[255, 1], [256], [257, 0, 3], [1] * 129, [5] * 700, [2047, 1, 2048, 2049], [0, 0]])
def test_product_tiles(lens, precision):
    """The standalone product at the edges of its tiles: one rounding per product
    and sum (FP32: of the value and of x), as in the parity tests of larger ones."""
    rng = np.random.default_rng(5)
    rows = np.repeat(np.arange(len(lens)), lens)
    cols = np.concatenate([np.sort(rng.choice(N, k, replace=False)) for k in lens]).astype(int)
    A = I.CSR.from_scipy(sp.csr_matrix((rng.standard_normal(cols.size), (rows, cols)), shape=(len(lens), N)))
    Q = I.CSR.from_scipy(sp.identity(N, format="csr"))
    sol = pdhcg.Solver(I.QP(Q, A, np.ones(len(lens)), np.zeros(N)), pdhcg.Settings(power_iters=1))
    x = rng.standard_normal(N)
    got = sol.spmv(1, x, precision=precision).cpu().numpy()
    ref = O.matvec(A, x)
    scale = O.matvec(I.CSR(A.nrows, A.ncols, A.rowptr, A.col, np.abs(A.val)), np.abs(x)) + 1e-300
    assert np.max(np.abs(got - ref) / scale) <= (2 * 2.0 ** -24 * 1.01 if precision else 1e-14)
    got = sol.spmv(2, np.arange(1.0, len(lens) + 1)).cpu().numpy()
    ref = O.matvec_t(A, np.arange(1.0, len(lens) + 1))
    assert np.max(np.abs(got - ref)) <= 1e-12 * max(1.0, np.abs(ref).max())
    sol.close()
