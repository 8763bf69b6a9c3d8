"""The warm-start network's matrix-product kernel at the edges of its tiles
(64 and 128 rows and columns, stages of 128 and steps of 32 along k, chunks of
the k range), against an FP64 evaluation of the same bfloat16 operands.

Inputs and weights are small integers, sparse enough that every hidden
activation is an integer below 256: the operands are then exact in bfloat16 and
every sum exact in FP32 whatever its order, so the outputs must equal the
reference bit for bit.  Gradients hold G = 2 (O - T) / count rounded to
bfloat16: a weight gradient is compared with the FP64 product of the same
rounded operands, with the bound of an FP32 sum of k products in any order,
k 2^-23 sum |a||b| (output layer), and where an operand was itself rounded to
bfloat16 from such a sum (hidden layers), one unit 2^-8 of it more."""
import numpy as np
import pytest

from oracle import mlp_oracle as M

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2405_16160_amd import mlp  # noqa: E402

# n_in, n_hid, n_out, batch
SIZES = [(1, 1, 1, 1), (31, 64, 63, 64), (32, 65, 64, 65), (33, 130, 129, 63), (129, 128, 257, 200), (20, 512, 66, 130),
         (7, 96, 1100, 33)]


def integer_net(rng, n_in, n_hid, n_out):
    """Weights in {-1, 0, 1} with about four non-zeros per output, integer biases."""
    out = []
    for a, b in ((n_in, n_hid), (n_hid, n_hid), (n_hid, n_out)):
        W = np.where(rng.uniform(size=(a, b)) < min(1.0, 4 / a), rng.integers(-1, 2, (a, b)), 0)
        out += [W.astype(np.float64), rng.integers(-2, 3, b).astype(np.float64)]
    return out


@pytest.mark.parametrize("n_in,n_hid,n_out,B", SIZES)
def test_products_at_tile_edges(n_in, n_hid, n_out, B):
    print(f"[mlp tiles] {n_in}-{n_hid}-{n_hid}-{n_out} batch {B}", flush=True)
    rng = np.random.default_rng([n_in, n_hid, n_out, B])
    params = integer_net(rng, n_in, n_hid, n_out)
    X = rng.integers(-2, 3, (B, n_in)).astype(np.float64)
    T = rng.integers(-3, 4, (B, n_out)).astype(np.float64)
    H = M.forward(params, X)
    assert max(np.abs(h).max() for h in H[1:3]) < 256
    net = mlp.Network(n_in, n_hid, n_out, max_batch=B, params=params)
    dev = lambda a: torch.tensor(a, dtype=torch.float32, device="cuda")  # noqa: E731
    assert np.array_equal(net.forward(dev(X)).cpu().numpy(), H[3].astype(np.float32))
    loss, grads = net.loss_grad(dev(X), dev(T), want_grads=True)
    net.close()
    assert loss == np.float32(np.mean((H[3] - T) ** 2))
    # the FP32 expression 2 d scale, then bfloat16
    d32 = (H[3] - T).astype(np.float32)
    G32 = np.float32(2.0) * d32 * np.float32(1.0 / (B * n_out))
    G = M.round_bf16(G32)
    u = 2.0 ** -23
    W2, W3 = params[2], params[4]

    def check(name, got, ref, bound):
        err = np.abs(got - ref) - bound
        assert np.all(err <= 0.0), (name, err.max())

    check("dW3", grads[4], H[2].T @ G, B * u * (H[2].T @ np.abs(G)))
    check("db3", grads[5], G32.astype(np.float64).sum(0), B * u * np.abs(G32).astype(np.float64).sum(0))
    D2 = (G @ W3.T) * (H[2] > 0)
    e2 = n_out * u * (np.abs(G) @ np.abs(W3.T)) * (H[2] > 0)
    check("db2", grads[3], D2.sum(0), (e2 + B * u * (np.abs(D2) + e2)).sum(0))
    r2 = e2 + 2.0 ** -8 * (np.abs(D2) + e2)
    check("dW2", grads[2], H[1].T @ D2, H[1].T @ (r2 + B * u * (np.abs(D2) + r2)))
    D1 = (D2 @ W2.T) * (H[1] > 0)
    e1 = ((r2 + n_hid * u * (np.abs(D2) + r2)) @ np.abs(W2.T)) * (H[1] > 0)
    check("db1", grads[1], D1.sum(0), (e1 + B * u * (np.abs(D1) + e1)).sum(0))
    r1 = e1 + 2.0 ** -8 * (np.abs(D1) + e1)
    check("dW1", grads[0], X.T @ D1, np.abs(X).T @ (r1 + B * u * (np.abs(D1) + r1)))


@pytest.mark.parametrize("rows,cap,n,n_pair,n_rest", [(1, 64, 3, 1, 1), (5000, 96, 1501, 203, 2497), (4100, 4100, 1, 0, 130),
                                                      (130, 7, 2, 33, 31)])
def test_start_points_over_passes_and_odd_columns(rows, cap, n, n_pair, n_rest):
    """predict_start over more rows than one pass of its workspace holds, with
    duals at scattered rows and column counts off every vector width; 5 000 x 4 201
    outputs take the 128 x 128 tiles, the others 64 x 64."""
    print(f"[mlp tiles] start points: {rows} rows, max_batch {cap}, columns {n} + {n_pair} + {n_rest}", flush=True)
    rng = np.random.default_rng([rows, cap, n])
    n_in, n_hid, n_out, m = 5, 64, n + n_pair + n_rest, 2 * n_pair + n_rest
    params = integer_net(rng, n_in, n_hid, n_out)
    X = rng.integers(-2, 3, (rows, n_in)).astype(np.float64)
    Z = M.forward(params, X)[3]
    mu, sd = rng.standard_normal(n_out), rng.uniform(0.5, 2.0, n_out)
    perm = rng.permutation(m).astype(np.int32)
    plus, minus, rest = perm[:n_pair], perm[n_pair:2 * n_pair], perm[2 * n_pair:]
    dev = lambda a, t: torch.tensor(np.ascontiguousarray(a), dtype=t, device="cuda")  # noqa: E731
    net = mlp.Network(n_in, n_hid, n_out, max_batch=cap, params=params)
    x0, y0 = net.predict_start(dev(X, torch.float32), dev(mu, torch.float64), dev(sd, torch.float64), n,
                               *(dev(p, torch.int32) for p in (plus, minus, rest)), m)
    net.close()
    V = Z * sd + mu
    Y = np.zeros((rows, m))
    Y[:, plus] = np.maximum(V[:, n:n + n_pair], 0.0)
    Y[:, minus] = np.maximum(-V[:, n:n + n_pair], 0.0)
    Y[:, rest] = np.maximum(V[:, n + n_pair:], 0.0)
    assert np.array_equal(x0.cpu().numpy(), V[:, :n])
    assert np.array_equal(y0.cpu().numpy(), Y)
