"""mlp_backward and mlp_dense_backward on small dyadic numbers: every product
and every sum, in whatever order, is exact in float32 (the sum of the terms'
sizes stays under 2^24 granules, which the test checks), so the results equal
float64's.  A row that is left out or taken twice changes them at any n."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    from paper_1908_07847_amd import mlp
    return mlp


def cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


def picks(g, values, *shape):
    return g.choice(np.array(values, np.float64), shape)


def row_sums(d, X, granule):
    """d^T X with the proof that float32 has it exactly."""
    assert np.max(np.abs(d).T @ np.abs(X)) < 2 ** 24 * granule
    for v in (d, X):
        assert np.array_equal(v.astype(np.float32), v)
    full = d.T @ X
    for r in (0, len(d) // 2, len(d) - 1):      # what one lost row would do
        assert not np.array_equal(full, full - np.outer(d[r], X[r]))
    return full


def same(name, got, ref):
    got = got.detach().cpu().numpy().reshape(ref.shape)
    assert np.array_equal(got, ref), (name, int(np.sum(got != ref)))


@pytest.mark.parametrize("n,d,h,k,act,mse", [
    (64, 33, 10, 3, "sigmoid", False),
    (511, 33, 16, 3, "tanh", False),
    (1024, 130, 20, 2, "sigmoid", True),     # three input tiles
    (2048, 48, 195, 4, "tanh", True),        # the most rows of the few-rows form ...
    (2049, 48, 195, 4, "tanh", False),       # ... and row ranges
    (300, 33, 700, 3, "sigmoid", False),
    (4096, 200, 70, 8, "tanh", True),        # four input tiles, more than four outputs
    (20000, 64, 256, 16, "tanh", False),
    (20001, 130, 70, 4, "sigmoid", False),
    (65536, 33, 16, 1, "sigmoid", True),     # 512 ranges of 128 rows
    (50000, 33, 256, 3, "sigmoid", False),
])
def test_backward(M, n, d, h, k, act, mse):
    print(f"exact backward n={n} {d}-{h}-{k} {act} {'mse' if mse else 'dY'}", flush=True)
    g = np.random.default_rng(n + h)
    X, W1, W2 = picks(g, [-2, -1, 1, 2], n, d), picks(g, [-1, 1], h, d), picks(g, [-1, 1], k, h)
    A = picks(g, [0, 0.5, -0.5], n, h) if act == "tanh" else picks(g, [0, 0.5], n, h)
    Y, T, dY = np.full((n, k), 0.5), picks(g, [0, 1, 1.5], n, k), picks(g, [-1, 1], n, k)
    theta = np.concatenate([W1.ravel(), np.zeros(h), W2.ravel(), np.zeros(k)]).astype(np.float32)
    net = M.Net(d, h, k, n, theta=theta, act=act)
    grads, dX, loss = net.backward(cuda(X), cuda(A), cuda(Y), dY=None if mse else cuda(dY),
                                   T=cuda(T) if mse else None, want_dx=True)
    torch.cuda.synchronize()
    scale = 2.0 / (n * k) if mse else 1.0       # a power of two
    up = scale * (Y - T) if mse else dY
    d2 = up * 0.25
    d1 = (d2 @ W2) * (1 - A * A if act == "tanh" else A * (1 - A))
    unit = scale / 32                           # up/2 . 1/4 . slopes of quarters
    ones = np.ones((n, 1))
    same("gW1", grads.W1, row_sums(d1, X, unit))
    same("gb1", grads.b1, row_sums(d1, ones, unit))
    same("gW2", grads.W2, row_sums(d2, A, unit))
    same("gb2", grads.b2, row_sums(d2, ones, unit))
    same("dX", dX, d1 @ W1)
    if mse:
        same("loss", loss, np.array([np.mean((Y - T) ** 2)]))


@pytest.mark.parametrize("n,din,dout,act,over", [
    (64, 64, 64, 1, False), (513, 130, 33, 0, False),
    (2048, 64, 195, 0, False), (2049, 64, 195, 1, False),     # both sides of the few-rows rule
    (3000, 130, 70, 0, False),                                # ragged input tiles, partials of every range
    (4100, 700, 40, 1, False), (2100, 2200, 20, 0, False),    # ranges limited by the workspace to five, to one
    (20000, 64, 256, 1, False), (100003, 20, 24, 0, False),
    (70000, 16, 16, 1, True),                                 # dX over dY: one range, folds inside a wave's rows
])
def test_dense_backward(M, n, din, dout, act, over):
    from paper_1908_07847_amd._lib import lib
    print(f"exact dense backward n={n} {din}->{dout} act={act}", flush=True)
    g = np.random.default_rng(n + dout)
    X, W = picks(g, [-2, -1, 1, 2], n, din), picks(g, [-1, 1], dout, din)
    Y = picks(g, [0, 0.5, -0.5], n, dout) if act else picks(g, [0.25, 0.5], n, dout)
    dY = picks(g, [-1, 1], n, dout)
    Xd, Yd, dYd, Wd = cuda(X), cuda(Y), cuda(dY), cuda(W)
    gW, gb = torch.empty_like(Wd), torch.empty(dout, device="cuda")
    dX = dYd if over else torch.empty_like(Xd)
    ws = torch.empty(n * dout, device="cuda")
    assert lib.mlp_dense_backward(Xd.data_ptr(), Yd.data_ptr(), dYd.data_ptr(), n, din, dout, Wd.data_ptr(), act,
                                  gW.data_ptr(), gb.data_ptr(), dX.data_ptr(), ws.data_ptr(), ws.numel() * 4, None) == 0
    torch.cuda.synchronize()
    dZ = dY * (1 - Y * Y if act else Y * (1 - Y))
    same("gW", gW, row_sums(dZ, X, 1 / 16))
    same("gb", gb, row_sums(dZ, np.ones((n, 1)), 1 / 16))
    same("dX", dX, dZ @ W)
