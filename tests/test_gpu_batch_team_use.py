"""That the batches of test_gpu_batch_teams.py are solved with teams at all (a refused
launch falls back to a workgroup per instance without an error), the adaptive step
with teams, and what the queries report.

Tolerances as there: 25 iterations that differ in the order of sums only, 1e-10 in
FP64 and 2e-5 with FP32 products.
"""
import numpy as np
import pytest

from paper_2405_16160_amd import instances as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2405_16160_amd import pdhcg  # noqa: E402
from test_gpu_batch_teams import ITERS, batch_of  # noqa: E402


@pytest.mark.parametrize("name", ["factored", "wide", "queue", "dense", "no_rows", "family"])
def test_teams_are_used(name):
    qps, factors = batch_of(name)
    print(f"[teams used] {name}", flush=True)
    b = pdhcg.Batch(qps, pdhcg.Settings(tol_rel_kkt=1e-14, max_iters=ITERS), lowrank=factors)
    planned, used = b.teams()
    assert planned > 0 and used == 0
    b.solve()
    assert b.teams() == (planned, planned)
    b.set_threads(512)
    b.solve()
    assert b.teams() == (planned, 0)
    b.close()


@pytest.mark.parametrize("precision", [0, 1])
def test_adaptive_step_with_teams(precision):
    qps = [I.random_qp(n=n, m=n // 2, r_rows=n // 2, q_density=0.02, a_density=0.02, family=22, instance=i)
           for i, n in enumerate((900, 40, 600, 333))]
    print(f"[teams adaptive] precision={precision}", flush=True)
    s = pdhcg.Settings(tol_rel_kkt=1e-14, max_iters=ITERS, cg_rule=1, max_cg_iters=3, precision=precision, step_rule=1)
    b = pdhcg.Batch(qps, s)
    out = {}
    for threads in (512, 256):
        b.set_threads(threads)
        x, y, rs = b.solve()
        assert all(r["iters"] == ITERS for r in rs)
        out[threads] = x.cpu().numpy().copy(), y.cpu().numpy().copy(), [r["rejected_steps"] for r in rs]
    assert b.teams()[1] > 0
    b.close()
    tol = 2e-5 if precision else 1e-10
    (x1, y1, j1), (x, y, j) = out[512], out[256]
    assert j == j1
    assert np.linalg.norm(x - x1) <= tol * np.linalg.norm(x1)
    assert np.linalg.norm(y - y1) <= tol * max(np.linalg.norm(y1), np.linalg.norm(x1))
