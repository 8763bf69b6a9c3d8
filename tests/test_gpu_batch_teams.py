"""Batches whose large instances get a team of workgroups.

A batch solved with teams (256 threads, co-resident launch with a queue for the
small instances) against the same batch with one workgroup per instance (512
threads: no teams), after a fixed number of iterations with a fixed number of CG
steps.  The two differ in the order of sums only: 25 iterations of products with
at most 2000 terms (2000 eps = 4e-13 each) grow by less than 1e2, so 1e-10 in FP64;
with FP32 products a changed last bit of x may round to another FP32 value, 2^-24 =
6e-8 per product, so 2e-5.
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

ITERS = 25


def batch_of(name):
    """(QPs, factors or None)"""
    if name == "factored":     # n, k at the chunk edges of the dense products; n = 9 stays a single
        sizes = [2000, 1025, 777, 130, 9]
    elif name == "wide":       # a factor of more than 256 columns, more rows than one staged operand
        sizes = [2610]
    elif name == "queue":      # one team and more singles than are resident
        sizes = [1500] + [24] * 700
    elif name == "dense":
        return [I.portfolio_qp(i, n=n) for i, n in enumerate((650, 257, 40))], None
    elif name == "no_rows":
        qps = [I.portfolio_qp(i, n=n) for i, n in enumerate((640, 512))]
        empty = lambda n: I.CSR(0, n, np.zeros(1, np.int64), np.zeros(0, np.int32), np.zeros(0))
        return [I.QP(q.Q, empty(q.n), np.zeros(0), q.c) for q in qps], None
    else:                      # members that share Q and A (and one launch for ||A||)
        fam = I.mpc_family(T=30, nx=12, nu=5)
        rng = np.random.default_rng(3)
        return [I.QP(fam.Q, fam.A, fam.b_for(0.1 * rng.standard_normal(fam.nx)), fam.c) for _ in range(7)], None
    made = [I.portfolio_lowrank(i, n=n) for i, n in enumerate(sizes)]
    return [q for q, _ in made], [f for _, f in made]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("name", ["factored", "wide", "queue", "dense", "no_rows", "family"])
def test_team_equals_one_workgroup(name, precision):
    qps, factors = batch_of(name)
    print(f"[teams] {name} precision={precision}", flush=True)
    s = pdhcg.Settings(tol_rel_kkt=1e-14, max_iters=ITERS, cg_rule=1, max_cg_iters=3, precision=precision,
                       ruiz_iters=4 if name == "factored" else 0)
    b = pdhcg.Batch(qps, s, lowrank=factors)
    out = {}
    for threads in (512, 256, 256):   # (the second with teams finds their barriers and queue used)
        b.set_threads(threads)
        x, y, rs = b.solve()
        assert all(r["iters"] == ITERS for r in rs)
        out.setdefault(threads, []).append((x.cpu().numpy().copy(), y.cpu().numpy().copy()))
    b.close()
    tol = 2e-5 if precision else 1e-10
    (x1, y1), = out[512]
    for x, y in out[256]:
        assert np.linalg.norm(x - x1) <= tol * np.linalg.norm(x1)
        assert np.linalg.norm(y - y1) <= tol * max(np.linalg.norm(y1), np.linalg.norm(x1))
    assert np.array_equal(out[256][0][0], out[256][1][0])
    assert np.array_equal(out[256][0][1], out[256][1][1])


def test_team_against_oracle():
    qps, _ = batch_of("family")
    b = pdhcg.Batch(qps, pdhcg.Settings(tol_rel_kkt=1e-6, max_iters=100_000))
    X, Y, rs = (v if isinstance(v, list) else v.cpu().numpy() for v in b.solve())
    for i, (qp, r) in enumerate(zip(qps, rs)):
        x, y = X[b.n_off[i]:b.n_off[i + 1]], Y[b.m_off[i]:b.m_off[i + 1]]
        ref = O.solve(qp, O.Settings(tol=1e-9, max_iters=400_000))
        assert r["status"] == 0
        assert O.kkt(qp, x, y)["rel_kkt"] <= 1e-6 * (1 + 1e-6)
        assert np.linalg.norm(x - ref.x) <= 1e-4 * np.linalg.norm(ref.x)
    b.close()


def test_shared_norm():
    """||A|| formed once for a family equals the oracle's and every member's own
    (100 steps of the power iteration, sums of at most 2000 terms: 1e-12)."""
    qps, _ = batch_of("family")
    s = pdhcg.Settings(tol_rel_kkt=1e-4, max_iters=3)
    shared = pdhcg.Batch(qps, s)
    rs = shared.solve()[2]
    A = qps[0].A
    copy = I.CSR(A.nrows, A.ncols, A.rowptr.copy(), A.col.copy(), A.val.copy())
    own = pdhcg.Batch(qps[:1] + [I.QP(qps[1].Q, copy, qps[1].b, qps[1].c)], s)   # two matrices: no sharing
    want = O.opnorm(A)
    for r in rs + own.solve()[2]:
        assert r["norm_A"] == pytest.approx(want, rel=1e-12)
    shared.close()
    own.close()
