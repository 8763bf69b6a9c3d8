"""Waits of the solver's kernels, on the CPU: the library built for the host with a
lane scheduler (tests/simt), so that a wave or a workgroup that runs ahead of the
others does so on every run.

What the kernels compute must not depend on that order: each case is solved with
the waves taken from the first to the last and from the last to the first, the
workgroups of a grid each running until it has to wait, and gives equal bits both
times; and in FP64 the oracle's counts and point (sums of at most 1200 terms,
1200 eps = 3e-13 each, growing by less than 1e2 over the few iterations: 1e-10).
"""
import ctypes

import numpy as np
import pytest

from oracle import oracle as O
from paper_2405_16160_amd import build, instances as I, pdhcg

from simt_host import build as build_host


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    """the host library behind the Python binding, device tensors on the CPU"""
    import torch
    with pytest.MonkeyPatch.context() as mp:
        cpu = torch.device("cpu")
        mp.setattr(build, "LIB", build_host(str(tmp_path_factory.mktemp("simt"))))
        mp.setattr(pdhcg, "_lib", None)
        mp.setattr(pdhcg, "_stream_ptr", lambda: None)
        mp.setattr(torch, "device", lambda *a: cpu)
        mp.setattr(torch.cuda, "current_device", lambda: 0)
        mp.setattr(torch.cuda, "synchronize", lambda: None)
        lib = pdhcg.lib()
        lib.simt_tick(100_000)   # (a wait that never ends: over after 5000 polls)
        yield lib
        lib.simt_tick(1)


def no_rows(n):
    return I.CSR(0, n, np.zeros(1, np.int64), np.zeros(0, np.int32), np.zeros(0))


def sparse_qp(m, long_row=False):
    """n = 60 (1200 with a row of A beyond 1024 entries), m rows"""
    if long_row:
        q = I.random_qp(n=1200, m=8, r_rows=30, q_density=0.01, a_density=0.01, family=21, instance=0)
        import scipy.sparse as sp
        rng = np.random.default_rng(5)
        M = sp.csr_matrix((q.A.val, q.A.col, q.A.rowptr), shape=(8, 1200)).tolil()
        M[3] = 0.1 * rng.standard_normal(1200)
        M = M.tocsr()
        A = I.CSR(8, 1200, M.indptr.astype(np.int64), M.indices.astype(np.int32), M.data)
        return I.QP(q.Q, A, q.b, q.c)
    q = I.random_qp(n=60, m=max(m, 1), r_rows=24, q_density=0.1, a_density=0.1, family=22, instance=m)
    return q if m else I.QP(q.Q, no_rows(60), np.zeros(0), q.c)


def both_orders(host, run):
    out = []
    for order in (0, 1):
        host.simt_wave_order(order)
        out.append(run())
    host.simt_wave_order(0)
    return out


def check(qp, settings, runs):
    """runs: (x, y, result) of each order"""
    (x, y, r), (x1, y1, r1) = runs
    drop = ("setup_s", "solve_s", "kernel_s")
    assert np.array_equal(x, x1) and np.array_equal(y, y1)
    assert all(r[k] == r1[k] for k in r if k not in drop), (r, r1)
    o = O.solve(qp, O.Settings(tol=settings.tol_rel_kkt, max_iters=settings.max_iters,
                               eval_period=settings.eval_period))
    assert (r["iters"], r["cg_iters_total"], r["restarts"]) == (o.iters, o.cg_steps, o.restarts)
    assert np.linalg.norm(x - o.x) <= 1e-10 * np.linalg.norm(o.x)
    assert np.linalg.norm(y - o.y) <= 1e-10 * (1 + np.linalg.norm(o.y))
    assert r["rel_kkt"] == pytest.approx(O.kkt(qp, x, y)["rel_kkt"], rel=1e-8)


CASES = {"m=0": (0, False), "m=1": (1, False), "m=24": (24, False), "long row": (8, True)}


@pytest.mark.parametrize("name", CASES)
def test_average_evaluation(host, name):
    """The restart evaluation reduces the average's n-side and m-side one after the
    other in the same stretch of LDS: solve kernel, batch kernel, and the batch
    kernel with a dense Q."""
    qp = sparse_qp(*CASES[name])
    s = pdhcg.Settings(tol_rel_kkt=1e-9, max_iters=20, eval_period=4, num_blocks=1)

    def single():
        h = pdhcg.Solver(qp, s)
        x, y, r = h.solve()
        return x.numpy().copy(), y.numpy().copy(), r

    check(qp, s, both_orders(host, single))
    check(qp, s, both_orders(host, lambda: pdhcg.solve_batch([qp], s)[0]))
    if qp.n == 60:
        full = I.portfolio_qp(3, n=60)
        full = I.QP(full.Q, qp.A, qp.b, qp.c)
        check(full, s, both_orders(host, lambda: pdhcg.solve_batch([full], s)[0]))


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("form", [1, 2])
def test_partials_of_the_next_phase(host, form, precision):
    """A workgroup that is through a barrier and on to its next partial sums while
    another has yet to read those of before: CG steps with one barrier each (form 1;
    FP32: the chained steps), and the point's residuals formed anew before a stop
    (FP32: certified) and at the iteration limit."""
    qp = sparse_qp(1)
    for tol, iters in ((1e-9, 12), (1e-1, 100)):
        s = pdhcg.Settings(tol_rel_kkt=tol, max_iters=iters, eval_period=4, num_blocks=2, cg_form=form,
                           precision=precision)

        def single():
            h = pdhcg.Solver(qp, s)
            x, y, r = h.solve()
            return x.numpy().copy(), y.numpy().copy(), r

        runs = both_orders(host, single)
        if precision == 0:
            check(qp, s, runs)
        else:   # (the oracle has no FP32 products: one workgroup's result, 2^-24 of each product, as above)
            s.num_blocks = 1
            x1, y1, r1 = single()
            x, y, r = runs[0]
            assert np.array_equal(x, runs[1][0]) and np.array_equal(y, runs[1][1])
            assert (r["status"], r["iters"], r["restarts"]) == (r1["status"], r1["iters"], r1["restarts"])
            assert np.linalg.norm(x - x1) <= 1e-4 * np.linalg.norm(x1)
            assert r["rel_kkt"] == pytest.approx(O.kkt(qp, x, y)["rel_kkt"], rel=1e-6)


@pytest.mark.parametrize("n1,n2", [(512, 0), (450, 60), (449, 1), (448, 64), (64, 448), (0, 512), (511, 1)])
def test_row_sums_stay_in_the_staging_area(host, n1, n2):
    """A row of [Q | A'] that fills its tile, summed by a wave, in the last stretch of
    the staging area: the surplus reads of the shorter part end inside it."""
    out = (ctypes.c_double * 2)()
    assert host.simt_row_sums(n1, n2, out) == 0
    assert list(out) == [n1, 1024.0 * n2]


def team_qps(shared):
    """a QP that gets a team of workgroups among others; shared: three with one Q and A"""
    if shared:
        fam = I.mpc_family(T=24, nx=10, nu=4)
        rng = np.random.default_rng(3)
        return [I.QP(fam.Q, fam.A, fam.b_for(0.1 * rng.standard_normal(fam.nx)), fam.c) for _ in range(3)]
    return [I.random_qp(n=n, m=n // 2, r_rows=n // 2, q_density=0.02, a_density=0.02, family=22, instance=i)
            for i, n in enumerate((700, 40, 300))]


def solve_handle(qps, s, threads=256):
    b = pdhcg.Batch(qps, s)
    b.set_threads(threads)
    x, y, rs = b.solve()
    out = x.numpy().copy(), y.numpy().copy(), rs, b.teams()
    b.close()
    return out


CAPPED = dict(tol_rel_kkt=1e-12, max_iters=5, eval_period=2, cg_rule=1, max_cg_iters=3, power_iters=20)


@pytest.mark.parametrize("fault", ["refuse", "late"])
@pytest.mark.parametrize("shared", [False, True])
def test_batch_without_its_teams(host, shared, fault):
    """The cooperative launches of a batch (the shared norm's, the teams') refused, or
    their barriers timing out: the batch is solved a workgroup per instance, to the
    512-thread result."""
    qps, s = team_qps(shared), pdhcg.Settings(**CAPPED)
    want = solve_handle(qps, s, threads=512)
    host.simt_launches()
    teams = solve_handle(qps, s)
    assert host.simt_launches() // 1000 == (2 if shared else 1)
    (host.simt_refuse if fault == "refuse" else host.simt_late)(4)
    plain = solve_handle(qps, s)
    host.simt_refuse(0)
    host.simt_late(0)
    # (the large QP or all three of the family; none with 512 threads or after the fault)
    n = 3 if shared else 1
    assert (want[3], teams[3], plain[3]) == ((n, 0), (n, n), (n, 0))
    for x, y, rs, _ in (teams, plain):
        assert [r["iters"] for r in rs] == [5] * 3
        for r, w in zip(rs, want[2]):
            assert r["norm_A"] == pytest.approx(w["norm_A"], rel=1e-12)
        assert np.linalg.norm(x - want[0]) <= 1e-10 * np.linalg.norm(want[0])
        assert np.linalg.norm(y - want[1]) <= 1e-10 * np.linalg.norm(want[0])


def test_time_limit_covers_the_second_launch(host):
    """A batch whose first launch ended in a barrier's time-out (5 s) is solved again
    within the same limit of 5.5 s, and kernel_s covers both launches."""
    qps, s = team_qps(False), pdhcg.Settings(**{**CAPPED, "time_limit_s": 5.5})
    host.simt_tick(1)
    host.simt_launches()
    host.simt_late(1)
    rs = solve_handle(qps, s)[2]
    host.simt_tick(100_000)
    assert host.simt_launches() == 1003   # the teams' launch; two that set up a launch and the one without teams
    assert [r["status_name"] for r in rs] == ["TIME_LIMIT"] * 3
    assert all(r["iters"] == 0 and r["kernel_s"] > 5.0 for r in rs)


def test_autotune_repeats_a_launch_that_timed_out(host):
    """A 256-thread repetition whose teams' barrier timed out is timed again without
    teams, not taken as it is: one launch with teams, then two pairs of the clock and a
    batch kernel, at 256 and at 512 threads."""
    b = pdhcg.Batch(team_qps(False), pdhcg.Settings(**CAPPED))
    host.simt_launches()
    host.simt_late(1)
    t = b.autotune(1)
    b.close()
    assert host.simt_launches() == 1005
    assert t["kernel_s"][256] < 5.0 and t["kernel_s"][512] < 5.0


@pytest.mark.parametrize("precision", [0, 1])
def test_streamed_kernels_equal_the_others(host, precision):
    """The 256-thread kernels with and without streamed matrices: equal bits.  (n = 60:
    streamed past an L2 of 320 bytes.)"""
    qp = sparse_qp(24)
    out = []
    for l2 in (320, 319):
        host.simt_l2(l2)
        h = pdhcg.Solver(qp, pdhcg.Settings(tol_rel_kkt=1e-9, max_iters=9, eval_period=4, num_blocks=2, threads=256,
                                            cg_form=2, precision=precision))
        x, y, r = h.solve()
        out.append((x.numpy().copy(), y.numpy().copy(), r["rel_kkt"], r["norm_A"]))
    host.simt_l2(4 << 20)
    (x, y, k, a), (x1, y1, k1, a1) = out
    assert np.array_equal(x, x1) and np.array_equal(y, y1) and (k, a) == (k1, a1)
