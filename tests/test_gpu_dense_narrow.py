"""Dense Q of at most 256 columns (rows split over the waves) and just above.

A few iterations with a fixed number of CG steps against the oracle's iterates:
sums of at most 258 terms, 258 eps = 6e-14, growing by less than 1e2 over 8
iterations of 3 CG steps, so 1e-10; FP32 values: 2^-24 = 6e-8 per product, so 2e-5.
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


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 128, 129, 192, 193, 255, 256, 257])
def test_dense_columns(n, precision):
    print(f"[dense] n={n} precision={precision}", flush=True)
    qp = I.portfolio_qp(0, n=n)
    ref = O.solve(qp, O.Settings(tol=1e-15, max_iters=8, cg_rule=1, max_cg=3))
    (x, y, r), = pdhcg.solve_batch([qp], pdhcg.Settings(tol_rel_kkt=1e-15, max_iters=8, cg_rule=1, max_cg_iters=3,
                                                        precision=precision))
    tol = 2e-5 if precision else 1e-10
    assert r["iters"] == ref.iters
    assert np.linalg.norm(x - ref.x) <= tol * np.linalg.norm(ref.x)
    assert np.linalg.norm(y - ref.y) <= tol * max(np.linalg.norm(ref.y), np.linalg.norm(ref.x))
