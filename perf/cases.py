"""Timed cases of the solver's public entry points.

Each case is one kind of work that a program built on this framework does:
a product with a matrix of a handle, a solve of one QP, a batched solve, and the
inference and training of the warm-start network.  ``listed()`` names one case
per kind and range, ``draw(rng)`` gives others of the same ranges,
``prepare(case, seed)`` makes what a program holds before the call,
``run(state)`` is one pass, ``work(case)`` the bytes and operations a pass
cannot do without, and ``exact(case, seed)`` the same outputs from plain FP64
torch code of this file.

Kinds and what they stand for:

* ``spmv``      a product with Q, A or A' of a handle (building a right-hand
                side or checking a residual with the library's own matrices);
* ``random``    one random sparse QP, n = 1e3 in FP64 to n = 1e5 with FP32
                products (the sizes of the two plain benchmark families);
* ``powerlaw``  one preconditioned power-law QP, up to n = 2e6, m = 1e6;
* ``lowrank``   one QP whose Q is given by a sparse factor;
* ``mpc``       one linear-MPC handle re-solved for a new initial state from
                the previous solution (set_b, then solve);
* ``portfolio`` a packed batch of preconditioned portfolio QPs, Q factored,
                n log-uniform in [50, 2000] (the headline workload's law);
* ``family``    a packed batch of linear-MPC members that share Q and A (the
                generation of training targets for the warm start);
* ``host``      the one-call batched solve of a few small dense portfolio QPs
                from host arrays;
* ``predict``   start points for members of a family from the trained network;
* ``train``     an epoch of training steps, loss and weights read at its end.

A solve ends at relKKT <= tol or at its iteration budget (``iters``), as a
program with a deadline sets it.  The MPC and small dense QPs run to tolerance;
the others run under a budget short enough that the iterates still follow from
the inputs: past about 200 iterations the inexact CG of an ill-conditioned Q
amplifies the last bit of a sum into another path to the same optimum.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2405_16160_amd import instances as I
from paper_2405_16160_amd import mlp, pdhcg

DEV = "cuda"


def listed():
    return [
        # the smallest call: one product with the tiny QP's Q, FP64
        dict(name="spmv_q_n1000_f64", kind="spmv", family="random", n=1000, m=500, which=0, precision=0),
        # the largest product: A of the power-law QP (row lengths 1 to 5000) with FP32 values
        dict(name="spmv_a_powerlaw_n2e6_f32", kind="spmv", family="powerlaw", n=2_000_000, m=1_000_000, which=1,
             precision=1),
        # the plain FP64 configuration: n = 1000, m = 500, 200 iterations
        dict(name="solve_random_n1000_f64", kind="random", n=1000, m=500, precision=0, tol=1e-6, iters=200,
             step_rule=0),
        # one large random sparse QP with FP32 products, 60 iterations
        dict(name="solve_random_n1e5_f32", kind="random", n=100_000, m=50_000, precision=1, tol=1e-6, iters=60,
             step_rule=0),
        # the largest QP: power-law rows, preconditioned, FP32 products, 40 iterations
        dict(name="solve_powerlaw_n2e6_f32", kind="powerlaw", n=2_000_000, m=1_000_000, precision=1, tol=1e-6,
             iters=40),
        # Q = P P' + diag(d) from its factor (the low-rank experiment's sizes), FP64, 60 iterations
        dict(name="solve_lowrank_n1e5_f64", kind="lowrank", n=100_000, m=50_000, k=10_000, precision=0, tol=1e-6,
             iters=60),
        # one MPC handle re-solved for a new initial state, warm, FP64 to 1e-4
        dict(name="solve_mpc_T50_f64", kind="mpc", T=50, nx=20, nu=10, precision=0, tol=1e-4, iters=100_000),
        # the headline batch's law at a size one launch holds resident
        dict(name="batch_portfolio_500_f32", kind="portfolio", count=500, nmin=50, nmax=2000, precision=1, tol=1e-4,
             iters=100),
        # targets for a learned warm start: members that share Q and A, FP64 to 1e-4
        dict(name="batch_mpc_600_f64", kind="family", count=600, T=50, nx=20, nu=10, precision=0, tol=1e-4,
             iters=100_000),
        # a few small QPs in one call from host arrays
        dict(name="batch_host_12_f64", kind="host", count=12, nmin=50, nmax=160, precision=0, tol=1e-4,
             iters=100_000),
        # start points for 4 000 family members (the held-out set of the learned warm start)
        dict(name="predict_4000x5500", kind="predict", rows=4000, n_in=20, n_hid=512, T=50, nx=20, nu=10, cap=256),
        # 16 training steps of 256 rows
        dict(name="train_16x256", kind="train", steps=16, batch=256, n_in=20, n_hid=512, n_out=5500, data=4096),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the listed ranges with sizes spread over them."""
    kind = rng.choice(["spmv", "random", "random", "powerlaw", "lowrank", "mpc", "portfolio", "family", "host",
                       "predict", "train"])
    if kind == "spmv":
        family = rng.choice(["random", "powerlaw"])
        n = _log_int(rng, 300, 100_000) if family == "random" else _log_int(rng, 20_000, 1_500_000)
        return dict(kind=kind, family=family, n=n, m=max(1, int(n * rng.uniform(0.3, 0.7))), which=rng.randrange(3),
                    precision=rng.randrange(2))
    if kind == "random":
        if rng.random() < 0.5:
            n = _log_int(rng, 100, 3000)
            rule = rng.choice([0, 0, 1])   # (the adaptive step is the more sensitive path: a shorter budget)
            return dict(kind=kind, n=n, m=max(1, n // 2 - rng.randrange(n // 10 + 1)), precision=0, tol=1e-6,
                        iters=rng.randrange(20, 40) if rule else rng.randrange(50, 200), step_rule=rule)
        n = _log_int(rng, 5_000, 150_000)
        return dict(kind=kind, n=n, m=n // 2 - rng.randrange(n // 10), precision=1, tol=1e-6,
                    iters=rng.randrange(15, 50), step_rule=0)
    if kind == "powerlaw":
        n = _log_int(rng, 30_000, 1_800_000)
        return dict(kind=kind, n=n, m=int(n * rng.uniform(0.3, 0.5)), precision=rng.randrange(2), tol=1e-6,
                    iters=rng.randrange(10, 40))
    if kind == "lowrank":
        n = _log_int(rng, 4_000, 100_000)
        return dict(kind=kind, n=n, m=n // 2 + rng.randrange(7), k=_log_int(rng, 300, 8_000), precision=0, tol=1e-6,
                    iters=rng.randrange(15, 60))
    if kind == "mpc":
        return dict(kind=kind, T=rng.randrange(10, 60), nx=rng.randrange(4, 21), nu=rng.randrange(1, 11), precision=0,
                    tol=1e-4, iters=100_000)
    if kind == "portfolio":
        return dict(kind=kind, count=rng.randrange(8, 400), nmin=50, nmax=_log_int(rng, 200, 1900), precision=1,
                    tol=1e-4, iters=rng.randrange(30, 100))
    if kind == "family":
        return dict(kind=kind, count=rng.randrange(16, 600), T=rng.randrange(10, 50), nx=rng.randrange(4, 21),
                    nu=rng.randrange(1, 11), precision=0, tol=1e-4, iters=100_000)
    if kind == "host":
        return dict(kind=kind, count=rng.randrange(1, 24), nmin=20, nmax=_log_int(rng, 40, 200), precision=0,
                    tol=1e-4, iters=100_000)
    if kind == "predict":
        return dict(kind=kind, rows=_log_int(rng, 1, 4000), n_in=rng.randrange(4, 41),
                    n_hid=rng.choice([64, 200, 256, 512]), T=rng.randrange(10, 51), nx=rng.randrange(4, 21),
                    nu=rng.randrange(1, 11), cap=rng.choice([64, 256, 1024]))
    return dict(kind="train", steps=rng.randrange(4, 17), batch=rng.choice([32, 100, 128, 256]),
                n_in=rng.randrange(4, 41), n_hid=rng.choice([64, 200, 256, 512]), n_out=_log_int(rng, 300, 5500),
                data=4096)


# ------------------------------------------------------------------- inputs


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) & 0x7FFFFFFF)


def _randn(g, *shape, dtype=torch.float64):
    return torch.randn(*shape, generator=g, device=DEV, dtype=dtype)


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device=DEV, dtype=torch.float64)


def _csr(rows, cols, vals, nrows, ncols):
    """instances.CSR of entries sorted by (row, column), from device tensors."""
    rowptr = torch.zeros(nrows + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(torch.bincount(rows, minlength=nrows), 0, out=rowptr[1:])
    return I.CSR(nrows, ncols, rowptr.cpu().numpy(), cols.to(torch.int32).cpu().numpy(), vals.cpu().numpy())


def _gaussian(g, nrows, ncols, density):
    """Sparse matrix with N(0, 1) values at about density * nrows * ncols uniform positions."""
    cnt = max(1, int(density * nrows * ncols))
    flat = torch.unique(torch.randint(nrows * ncols, (cnt,), generator=g, device=DEV))
    return _csr(flat // ncols, flat % ncols, _randn(g, flat.numel()), nrows, ncols)


def _symmetric(i, j, v, n):
    """The symmetric matrix with the sums of v at (i, j), i <= j, mirrored."""
    key, inv = torch.unique(torch.minimum(i, j) * n + torch.maximum(i, j), return_inverse=True)
    order = torch.argsort(inv, stable=True)          # sums in a fixed order
    s = torch.segment_reduce(v[order], "sum", lengths=torch.bincount(inv, minlength=key.numel()))
    a, b = key // n, key % n
    off = a != b
    full = torch.cat([key, b[off] * n + a[off]])
    val = torch.cat([s, s[off]])
    full, order = torch.sort(full)
    return _csr(full // n, full % n, val[order], n, n)


def _rhs(g, A):
    """c ~ N(0, 1) and b = A x0 + U[0, 1] with x0 ~ N(0, 1)."""
    c, x0 = _randn(g, A.ncols).cpu().numpy(), _randn(g, A.ncols).cpu().numpy()
    return A.to_scipy() @ x0 + _rand(g, A.nrows).cpu().numpy(), c


def _random_qp(g, n, m):
    """Q = R'R + 1e-2 I: about 5 entries per row of R at n = 1000 (density
    1e-2) down to 2 at n = 1e5 (2e-5), A 10 to 20 entries per row, the two
    plain families' laws at their sizes."""
    t = min(1.0, max(0.0, math.log(n / 1000) / math.log(100)))
    r, a = 10 * 0.2 ** t / n, 10 * 2.0 ** t / n
    R = _gaussian(g, max(1, n // 2), n, r).to_scipy()
    Q = I._symmetrize(R.T @ R + 1e-2 * I.sp.identity(n, format="csr"))
    A = _gaussian(g, m, n, a)
    b, c = _rhs(g, A)
    return I.QP(I.CSR.from_scipy(Q), A, b, c)


def _powerlaw_qp(g, n, m):
    """A with Pareto(1.5) row lengths in [1, 5000], mean about 8, uniform
    columns; Q = diag(U[0.01, 1]) + signed edges, about 5 entries per row."""
    u = 1.0 - _rand(g, m)
    L = torch.clamp(torch.round(2.75 * u ** (-1.0 / 1.5)), 1, min(5000, n)).to(torch.int64)
    row = torch.repeat_interleave(torch.arange(m, device=DEV), L)
    flat = torch.unique(row * n + torch.randint(n, (row.numel(),), generator=g, device=DEV))
    A = _csr(flat // n, flat % n, _randn(g, flat.numel()), m, n)
    i = torch.randint(n, (2 * n,), generator=g, device=DEV)
    j = torch.randint(n - 1, (2 * n,), generator=g, device=DEV)
    j = torch.where(j >= i, j + 1, j)
    w = _randn(g, 2 * n).abs()
    s = torch.where(_rand(g, 2 * n) < 0.5, -1.0, 1.0)
    d = torch.arange(n, device=DEV)
    Q = _symmetric(torch.cat([i, j, i, d]), torch.cat([i, j, j, d]), torch.cat([w, w, s * w, 0.01 + 0.99 * _rand(g, n)]), n)
    b, c = _rhs(g, A)
    return I.QP(Q, A, b, c)


def _lowrank_qp(g, n, m, k):
    """P with density 1e-3 (at least one entry per row), d ~ U[0.01, 0.1], A at density 1e-4 (at least 4 per row)."""
    flat = torch.randint(n * k, (int(1e-3 * n * k) + 1,), generator=g, device=DEV)
    one = torch.arange(n, device=DEV) * k + torch.randint(k, (n,), generator=g, device=DEV)
    flat = torch.unique(torch.cat([flat, one]))
    P = _csr(flat // k, flat % k, _randn(g, flat.numel()), n, k)
    d = (0.01 + 0.09 * _rand(g, n)).cpu().numpy()
    A = _gaussian(g, m, n, max(1e-4, 4.0 / n))
    b, c = _rhs(g, A)
    empty = I.CSR(n, n, np.zeros(n + 1, np.int64), np.zeros(0, np.int32), np.zeros(0))
    return I.QP(empty, A, b, c), P, d


def _portfolio(g, n, dense):
    """One portfolio QP: the dense Q, or a placeholder and its factor (F, d)."""
    k = int(math.ceil(n / 10))
    F = (_randn(g, n, k) / math.sqrt(n)).cpu().numpy()
    d = (0.01 + 0.09 * _rand(g, n)).cpu().numpy()
    c = -(0.05 + 0.02 * _randn(g, n)).cpu().numpy()
    A, b = I._portfolio_rows(n)
    if dense:
        Q = F @ F.T
        Q = 0.5 * (Q + Q.T)
        Q[np.diag_indices(n)] += d
        Qc = I.CSR(n, n, np.arange(0, n * n + 1, n, dtype=np.int64), np.tile(np.arange(n, dtype=np.int32), n), Q.ravel())
    else:
        Qc = I.CSR(n, n, np.arange(n + 1, dtype=np.int64), np.arange(n, dtype=np.int32), np.ones(n))
    return I.QP(Qc, A, b, c), (F, d)


def _portfolio_sizes(case):
    """Sizes log-spaced over [nmin, nmax], the same for every seed."""
    cnt = case["count"]
    t = (np.arange(cnt) + 0.5) / cnt
    return [int(round(case["nmin"] * (case["nmax"] / case["nmin"]) ** v)) for v in t]


def _states(g, fam, count):
    """Initial states x ~ N(0, I), shrunk into the ball that keeps u = 0 feasible."""
    x = _randn(g, count, fam.nx).cpu().numpy()
    r = np.linalg.norm(x, axis=1, keepdims=True)
    return x * np.minimum(1.0, fam.x_max / 0.95 * 0.999 / r)


def _settings(case, **more):
    return pdhcg.Settings(tol_rel_kkt=case["tol"], max_iters=case["iters"], precision=case["precision"], **more)


PRE = dict(ruiz_iters=10, pock_chambolle=1)


def _mlp_data(g, case, n_out, rows):
    """Standardised inputs, targets and He-uniform weights (packed)."""
    a, d = case["n_in"], case["n_hid"]
    parts = []
    for i, o in ((a, d), (d, d), (d, n_out)):
        parts += [((_rand(g, i, o) * 2 - 1) * math.sqrt(6.0 / i)).reshape(-1), torch.zeros(o, device=DEV, dtype=torch.float64)]
    w = torch.cat(parts).float()
    X = _randn(g, rows, a, dtype=torch.float32)
    return X, w


def _inputs(case, seed):
    """The case's problem data (host CSR and device tensors), from the seed alone."""
    g, kind = _gen(seed), case["kind"]
    if kind == "spmv":
        make = _random_qp if case["family"] == "random" else _powerlaw_qp
        qp = make(g, case["n"], case["m"])
        return dict(qp=qp, v=_randn(g, qp.m if case["which"] == 2 else qp.n))
    if kind == "random":
        return dict(qp=_random_qp(g, case["n"], case["m"]))
    if kind == "powerlaw":
        return dict(qp=_powerlaw_qp(g, case["n"], case["m"]))
    if kind == "lowrank":
        qp, P, d = _lowrank_qp(g, case["n"], case["m"], case["k"])
        return dict(qp=qp, P=P, d=d)
    if kind in ("mpc", "family"):
        fam = I.mpc_family(case["T"], case["nx"], case["nu"])
        cnt = 2 if kind == "mpc" else case["count"]
        return dict(fam=fam, bs=[fam.b_for(x) for x in _states(g, fam, cnt)])
    if kind in ("portfolio", "host"):
        made = [_portfolio(g, n, kind == "host") for n in _portfolio_sizes(case)]
        return dict(qps=[q for q, _ in made], factors=[f for _, f in made])
    if kind == "predict":
        fam_n, e, box = case["T"] * (case["nu"] + case["nx"]), case["T"] * case["nx"], 2 * case["T"] * (case["nu"] + case["nx"])
        n_out = fam_n + e + box
        X, w = _mlp_data(g, case, n_out, case["rows"])
        idx = torch.arange(2 * e + box, device=DEV, dtype=torch.int32)
        return dict(X=X, w=w, n=fam_n, m=2 * e + box, n_out=n_out, mu=0.1 * _randn(g, n_out), sd=0.05 + _rand(g, n_out),
                    plus=idx[:e].contiguous(), minus=idx[e:2 * e].contiguous(), rest=idx[2 * e:].contiguous())
    X, w = _mlp_data(g, case, case["n_out"], case["data"])
    T = _randn(g, case["data"], case["n_out"], dtype=torch.float32)
    perm = torch.randperm(case["data"], generator=g, device=DEV).to(torch.int32)
    return dict(X=X, w=w, T=T, rows=perm)


def prepare(case, seed):
    s, kind = _inputs(case, seed), case["kind"]
    s["case"] = case
    if kind == "spmv":
        s["solver"] = pdhcg.Solver(s["qp"], pdhcg.Settings(precision=case["precision"], power_iters=1))
        s["out"] = torch.empty(s["qp"].m if case["which"] == 1 else s["qp"].n, dtype=torch.float64, device=DEV)
    elif kind == "random":
        s["solver"] = pdhcg.Solver(s["qp"], _settings(case, step_rule=case["step_rule"]))
    elif kind == "powerlaw":
        s["solver"] = pdhcg.Solver(s["qp"], _settings(case, **PRE))
    elif kind == "lowrank":
        s["solver"] = pdhcg.Solver(s["qp"], _settings(case), lowrank=(s["P"], s["d"]))
    elif kind == "mpc":
        fam = s["fam"]
        s["solver"] = pdhcg.Solver(I.QP(fam.Q, fam.A, s["bs"][0], fam.c), _settings(case, warm_fallback=0))
        s["x0"], s["y0"], _ = s["solver"].solve()
    elif kind == "portfolio":
        s["batch"] = pdhcg.Batch(s["qps"], _settings(case, **PRE), lowrank=s["factors"])
    elif kind == "family":
        fam = s["fam"]
        s["batch"] = pdhcg.Batch([I.QP(fam.Q, fam.A, b, fam.c) for b in s["bs"]], _settings(case, warm_fallback=0))
    elif kind == "predict":
        s["net"] = mlp.Network(case["n_in"], case["n_hid"], s["n_out"], max_batch=case["cap"], params=s["w"].cpu().numpy())
    elif kind == "train":
        s["net"] = mlp.Network(case["n_in"], case["n_hid"], case["n_out"], max_batch=case["batch"],
                               params=s["w"].cpu().numpy())
        s["weights"] = torch.empty(s["net"].np, dtype=torch.float32, pin_memory=True)
    return s


def run(state):
    case, kind = state["case"], state["case"]["kind"]
    if kind == "spmv":
        return state["solver"].spmv(case["which"], state["v"], precision=case["precision"], out=state["out"])
    if kind in ("random", "powerlaw", "lowrank"):
        x, y, r = state["solver"].solve()
        return {"x": x, "y": y, "objective": r["primal_obj"]}
    if kind == "mpc":
        state["solver"].set_b(state["bs"][1])
        x, y, r = state["solver"].solve(x0=state["x0"], y0=state["y0"])
        return {"x": x, "y": y, "objective": r["primal_obj"]}
    if kind in ("portfolio", "family"):
        x, y, rs = state["batch"].solve()
        return {"x": x, "y": y, "objective": np.array([r["primal_obj"] for r in rs])}
    if kind == "host":
        outs = pdhcg.solve_batch(state["qps"], _settings(case, **PRE))
        return {"x": np.concatenate([o[0] for o in outs]), "y": np.concatenate([o[1] for o in outs]),
                "objective": np.array([o[2]["primal_obj"] for o in outs])}
    if kind == "predict":
        x0, y0 = state["net"].predict_start(state["X"], state["mu"], state["sd"], state["n"], state["plus"],
                                            state["minus"], state["rest"], state["m"])
        return {"x0": x0, "y0": y0}
    net, b = state["net"], case["batch"]
    for k in range(case["steps"]):
        at = (k * b) % (case["data"] - b + 1)
        net.train_rows(state["X"], state["T"], state["rows"][at:at + b], b, lr=1e-3)
    loss, steps = net.take_loss()
    pdhcg.lib().pdhcg_mlp_get_params(net.h, state["weights"].data_ptr())
    return {"weights": state["weights"], "loss": loss / steps}


# --------------------------------------------------------------------- work


def _shape(case):
    """(n, m, entries of Q or of its factors, entries of A) of a QP case, as expected."""
    kind = case["kind"]
    if kind in ("mpc", "family"):
        T, nx, nu = case["T"], case["nx"], case["nu"]
        return (T * (nx + nu), 2 * T * nx + 2 * T * (nx + nu), T * (nu + nx * nx),
                2 * T * nx * (1 + nu + nx) + 2 * T * (nx + nu))
    n, m = case["n"], case["m"]
    if kind == "lowrank":
        return n, m, 2 * (1e-3 * n * case["k"] + n), m * max(1e-4 * n, 4.0)
    if case.get("family", kind) == "powerlaw":
        return n, m, 5 * n, 8 * m
    t = min(1.0, max(0.0, math.log(n / 1000) / math.log(100)))
    return n, m, n * (1 + 0.5 * (10 * 0.2 ** t) ** 2 * min(1.0, 100 / n + 0.9)), m * 10 * 2.0 ** t


def work(case):
    """Inputs read once, outputs written once; operations: 2 per entry of every
    product that an iteration needs (one with Q, one with A, one with A' at
    least; about 500 iterations where the budget does not bind)."""
    kind = case["kind"]
    v = 4 if case.get("precision") else 8
    if kind == "spmv":
        n, m, nq, na = _shape(case)
        e, r, c = ((nq, n, n), (na, m, n), (na, n, m))[case["which"]]
        return dict(bytes=e * (v + 4) + 4 * (r + 1) + c * v + 8 * r, flops=2 * e)
    its = min(case.get("iters", 0), 500)
    if kind in ("random", "powerlaw", "lowrank", "mpc"):
        n, m, nq, na = _shape(case)
        return dict(bytes=12 * (nq + na) + 16 * (n + m), flops=its * (2 * nq + 4 * na))
    if kind == "family":
        n, m, nq, na = _shape(case)
        return dict(bytes=12 * (nq + na) + 16 * case["count"] * (n + m), flops=case["count"] * its * (2 * nq + 4 * na))
    if kind in ("portfolio", "host"):
        q = sum(n * math.ceil(n / 10) if kind == "portfolio" else n * n for n in _portfolio_sizes(case))
        n = sum(_portfolio_sizes(case))
        return dict(bytes=v * q + 8 * 10 * n, flops=its * (2 * q * (2 if kind == "portfolio" else 1) + 12 * n))
    a, d = case["n_in"], case["n_hid"]
    if kind == "predict":
        nv, m = case["T"] * (case["nu"] + case["nx"]), case["T"] * (2 * case["nu"] + 4 * case["nx"])
        o, B = nv + m - case["T"] * case["nx"], case["rows"]
        return dict(bytes=4 * (B * a + a * d + d * d + d * o) + 8 * B * (nv + m), flops=2 * B * (a * d + d * d + d * o))
    o, B, k = case["n_out"], case["batch"], case["steps"]
    w = a * d + d * d + d * o
    return dict(bytes=k * (4 * B * (a + o) + 4 * 6 * w) + 4 * w, flops=k * 6 * B * w)


# -------------------------------------------------------------------- exact


def _sparse(M):
    return torch.sparse_csr_tensor(torch.as_tensor(M.rowptr, device=DEV), torch.as_tensor(M.col, device=DEV).long(),
                                   torch.as_tensor(M.val, device=DEV), size=(M.nrows, M.ncols))


class _Op:
    """A CSR matrix as FP64 torch: products, its transpose's and the preconditioning statistics."""

    def __init__(self, M):
        self.M, self.S, self.T = M, _sparse(M), _sparse(I.CSR.from_scipy(M.to_scipy().T))
        self.rows = torch.repeat_interleave(torch.arange(M.nrows, device=DEV), torch.as_tensor(np.diff(M.rowptr), device=DEV))
        self.cols = torch.as_tensor(M.col, device=DEV).long()
        self.vals = torch.as_tensor(M.val, device=DEV)

    def stats(self, dim, scale_r, scale_c, mode):
        a = (self.vals * scale_r[self.rows] * scale_c[self.cols]).abs()
        n, at = (self.M.nrows, self.rows) if dim == 0 else (self.M.ncols, self.cols)
        return torch.zeros(n, device=DEV, dtype=torch.float64).scatter_reduce(0, at, a, "amax" if mode == 0 else "sum")


def _precondition(Q, A):
    """(D2, D1): 10 Ruiz steps and one Pock-Chambolle step on [[Q, A'], [A, 0]]."""
    d2, d1 = (torch.ones(k, device=DEV, dtype=torch.float64) for k in (A.M.ncols, A.M.nrows))
    for mode in [0] * 10 + [1]:
        q, t, a = Q.stats(0, d2, d2, mode), A.stats(1, d1, d2, mode), A.stats(0, d1, d2, mode)
        v = torch.maximum(q, t) if mode == 0 else q + t
        d2 = d2 / torch.where(v > 0, v, 1.0).sqrt()
        d1 = d1 / torch.where(a > 0, a, 1.0).sqrt()
    return d2, d1


def _solve_exact(qmul, amul, tmul, b, c, case, d2=None, d1=None):
    """Restarted PDHCG (Alg. 1 with the rules of Sec. 4) in FP64 torch from
    (0, 0): (x, y, objective) of the caller's problem."""
    n, m = c.numel(), b.numel()
    one = lambda k: torch.ones(k, device=DEV, dtype=torch.float64)  # noqa: E731
    D2, D1 = (one(n), one(m)) if d2 is None else (d2, d1)
    Q = lambda v: D2 * qmul(D2 * v)  # noqa: E731
    A = lambda v: D1 * amul(D2 * v)  # noqa: E731
    T = lambda v: D2 * tmul(D1 * v)  # noqa: E731
    bn, cn = float(b.abs().max()), float(c.abs().max())
    b, c = D1 * b, D2 * c
    v = 0.5 + ((torch.arange(n, device=DEV, dtype=torch.int64) * 40503) % 1024).double() / 1024.0
    v, lam = v / v.norm(), 0.0
    for _ in range(100):
        w = T(A(v))
        lam = float(w.norm())
        v = w / lam
    eta, omega = 0.5 / math.sqrt(lam), 1.0
    z = lambda k: torch.zeros(k, device=DEV, dtype=torch.float64)  # noqa: E731
    x, y, ax, xa, ya, x_anc, y_anc = z(n), z(m), z(m), z(n), z(m), z(n), z(m)
    k = total = 0
    eps, K_anchor, K_prev = 0.0, None, math.inf

    def kkt(x, y, u):
        Qx, Ty = Q(x), T(y)
        g = Qx + Ty + c
        xqx, cx, by = (float(t) for t in (x @ Qx, c @ x, b @ y))
        mx = lambda t: float(t.max())  # noqa: E731
        rp = mx(torch.clamp(u - b, min=0) / D1) / (1 + max(mx((u / D1).abs()), bn))
        rd = mx((g / D2).abs()) / (1 + max(mx((Qx / D2).abs()), mx((Ty / D2).abs()), cn))
        rg = abs(xqx + cx + by) / (1 + max(abs(0.5 * xqx + cx), abs(0.5 * xqx + by)))
        return max(rp, rd, rg), g, 0.5 * xqx + cx

    while True:
        kc, g, obj = kkt(x, y, ax)
        K_anchor = kc if K_anchor is None else K_anchor
        if kc <= case["tol"]:
            return D2 * x, D1 * y, obj
        ka = None
        if k > 0 and k % 64 == 0:
            au = A(xa)
            ka, _, obj_a = kkt(xa, ya, au)
            if ka <= case["tol"]:
                return D2 * xa, D1 * ya, obj_a
            Kc = min(ka, kc)
            why = Kc <= 0.2 * K_anchor or (Kc <= 0.8 * K_anchor and Kc > K_prev) or k >= 0.2 * total
            K_prev = Kc
            if why:
                moved = ka < kc
                if moved:
                    x, y, ax = xa.clone(), ya.clone(), au
                dx, dy = float((x - x_anc).norm()), float((y - y_anc).norm())
                if dx > 1e-10 and dy > 1e-10:
                    omega = math.exp(0.2 * math.log(dy / dx) + 0.8 * math.log(omega))
                x_anc, y_anc, xa, ya = x.clone(), y.clone(), x.clone(), y.clone()
                K_anchor, K_prev, k, eps, ka = Kc, math.inf, 0, 0.0, None
                if moved:
                    continue
        if total >= case["iters"]:
            if k > 0 and ka is None:
                ka, _, obj_a = kkt(xa, ya, A(xa))
            return (D2 * xa, D1 * ya, obj_a) if ka is not None and ka < kc else (D2 * x, D1 * y, obj)
        eps += 0.05 * kc
        tau, sigma = eta / omega, eta * omega
        r = -g
        rho, p = float(r @ r), r
        for l in range(100):
            if not rho > 0:
                break
            q = Q(p) + p / tau
            alpha = rho / float(p @ q)
            x = x + alpha * p
            r = r - alpha * q
            new = float(r @ r)
            if tau * math.sqrt(new) <= eps:
                break
            p, rho = r + (new / rho) * p, new
        u = A(x)
        y = torch.clamp(y + sigma * (2 * u - ax - b), min=0)
        ax = u
        xa = xa + (x - xa) / (k + 1)
        ya = ya + (y - ya) / (k + 1)
        k, total = k + 1, total + 1


def _dev(a):
    return torch.as_tensor(a, dtype=torch.float64, device=DEV)


def exact(case, seed):
    """The outputs of run() in FP64 torch; None where that takes too long
    (large batches) or follows the adaptive step's trials."""
    kind = case["kind"]
    if kind in ("family", "portfolio", "mpc") or case.get("step_rule"):
        return None
    s = _inputs(case, seed)
    if kind == "spmv":
        M = s["qp"].Q if case["which"] == 0 else s["qp"].A
        return (_Op(M).T if case["which"] == 2 else _sparse(M)) @ s["v"]
    if kind in ("random", "powerlaw", "lowrank"):
        qp, A = s["qp"], _Op(s["qp"].A)
        d2 = d1 = None
        if kind == "lowrank":
            P, d = _Op(s["P"]), _dev(s["d"])
            qmul = lambda v: P.S @ (P.T @ v) + d * v  # noqa: E731
        else:
            Q = _Op(qp.Q)
            qmul = lambda v: Q.S @ v  # noqa: E731
            if kind == "powerlaw":
                d2, d1 = _precondition(Q, A)
        x, y, obj = _solve_exact(qmul, lambda v: A.S @ v, lambda v: A.T @ v, _dev(qp.b), _dev(qp.c), case, d2, d1)
        return {"x": x, "y": y, "objective": obj}
    if kind == "host":
        outs = []
        for qp in s["qps"]:
            Qd, A = _Op(qp.Q), _Op(qp.A)
            d2, d1 = _precondition(Qd, A)
            D = _dev(qp.Q.to_scipy().toarray())
            Ad = _dev(qp.A.to_scipy().toarray())
            outs.append(_solve_exact(lambda v: D @ v, lambda v: Ad @ v, lambda v: Ad.T @ v, _dev(qp.b), _dev(qp.c), case, d2, d1))
        return {"x": torch.cat([o[0] for o in outs]), "y": torch.cat([o[1] for o in outs]),
                "objective": _dev([o[2] for o in outs])}
    a, d = case["n_in"], case["n_hid"]
    o = s["n_out"] if kind == "predict" else case["n_out"]
    sizes = [a * d, d, d * d, d, d * o, o]
    shapes = [(a, d), (d,), (d, d), (d,), (d, o), (o,)]
    W = [p.reshape(q) for p, q in zip(torch.split(s["w"].double(), sizes), shapes)]

    def net(X):
        h1 = torch.clamp(X @ W[0] + W[1], min=0)
        h2 = torch.clamp(h1 @ W[2] + W[3], min=0)
        return h1, h2, h2 @ W[4] + W[5]

    if kind == "predict":
        z = net(s["X"].double())[2] * s["sd"] + s["mu"]
        n, e = s["n"], s["plus"].numel()
        lam = z[:, n:n + e]
        return {"x0": z[:, :n], "y0": torch.clamp(torch.cat([lam, -lam, z[:, n + e:]], 1), min=0)}
    m1, m2, total = [torch.zeros_like(w) for w in W], [torch.zeros_like(w) for w in W], 0.0
    for k in range(case["steps"]):
        at = (k * case["batch"]) % (case["data"] - case["batch"] + 1)
        rows = s["rows"][at:at + case["batch"]].long()
        X, T = s["X"][rows].double(), s["T"][rows].double()
        h1, h2, out = net(X)
        total += float(((out - T) ** 2).mean())
        G = 2 * (out - T) / out.numel()
        D2 = (G @ W[4].T) * (h2 > 0)
        D1 = (D2 @ W[2].T) * (h1 > 0)
        grads = [X.T @ D1, D1.sum(0), h1.T @ D2, D2.sum(0), h2.T @ G, G.sum(0)]
        for i, gr in enumerate(grads):
            m1[i] = 0.9 * m1[i] + 0.1 * gr
            m2[i] = 0.999 * m2[i] + 0.001 * gr * gr
            W[i] = W[i] - 1e-3 * (m1[i] / (1 - 0.9 ** (k + 1))) / ((m2[i] / (1 - 0.999 ** (k + 1))).sqrt() + 1e-8)
    return {"weights": torch.cat([w.reshape(-1) for w in W]), "loss": total / case["steps"]}
