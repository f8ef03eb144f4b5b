"""The gradient kernels of mlp_backward and mlp_dense_backward against
float64 at the edges of their 64 x 64 tiles, row sets and row ranges.

Bounds: a sum of n float32 products in any order is within n u sum|terms| of
the exact one (u = 2^-24); a delta carries K + 8 further roundings, relative
to its own sum of |terms|."""
import sys

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
U = 2.0 ** -24


@pytest.fixture(scope="module")
def M():
    from paper_1908_07847_amd import mlp
    return mlp


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def within(name, got, ref, mag, terms):
    err = np.abs(got.detach().cpu().numpy().astype(np.float64).reshape(ref.shape) - ref)
    bound = terms * U * mag + 1e-30
    worst = float(np.max(err / bound))
    assert worst <= 1.0, (name, worst)


@pytest.mark.parametrize("n,d,h,k,act,mse", [
    (1, 1, 1, 1, "sigmoid", True),        # one of everything
    (31, 64, 64, 3, "sigmoid", False),    # one tile exactly, a short row set
    (129, 65, 65, 4, "tanh", True),       # one past every tile edge, five row sets
    (512, 33, 16, 3, "sigmoid", True),    # the most rows of a single range
    (513, 33, 16, 3, "sigmoid", False),   # ... and the fewest of several
    (3001, 20, 100, 5, "tanh", False),    # more than four outputs, ragged ranges
    (20000, 64, 256, 16, "sigmoid", True),
])
def test_backward_edges(M, n, d, h, k, act, mse):
    say(f"backward n={n} {d}-{h}-{k} {act} {'mse' if mse else 'dY'}")
    g = np.random.default_rng(n + h)
    X = g.normal(size=(n, d)).astype(np.float32)
    A = g.uniform(0.01, 0.99, (n, h)).astype(np.float32)
    Y = g.uniform(0.01, 0.99, (n, k)).astype(np.float32)
    T = (g.random((n, k)) < 0.3).astype(np.float32)
    dY = g.normal(size=(n, k)).astype(np.float32)
    theta = g.uniform(-0.5, 0.5, d * h + h + h * k + k).astype(np.float32)
    net = M.Net(d, h, k, n, theta=theta, act=act)
    grads, dX, loss = net.backward(cuda(X), cuda(A), cuda(Y), dY=None if mse else cuda(dY),
                                   T=cuda(T) if mse else None, want_dx=True)
    torch.cuda.synchronize()
    W1 = theta[:d * h].reshape(h, d).astype(np.float64)
    W2 = theta[d * h + h:d * h + h + k * h].reshape(k, h).astype(np.float64)
    X, A, Y = X.astype(np.float64), A.astype(np.float64), Y.astype(np.float64)
    up = 2.0 * (Y - T) / (n * k) if mse else dY.astype(np.float64)
    d2 = up * Y * (1 - Y)
    sl = 1 - A * A if act == "tanh" else A * (1 - A)
    d1, d1m = (d2 @ W2) * sl, (np.abs(d2) @ np.abs(W2)) * sl
    t = n + k + 8
    # Y - T is one rounding of a difference of numbers of size 1
    d2m = np.abs(d2) + (2.0 / (n * k) * Y * (1 - Y) if mse else 0.0)
    d1m = d1m + (d2m @ np.abs(W2)) * sl
    # 1 - A A (and 1 - A) round to u of 1, not of the difference
    d1m = d1m + (np.abs(d2) @ np.abs(W2)) * np.maximum(A, 1.0 - sl)
    d2m = d2m + np.abs(up) * Y
    within("gW1", grads.W1, d1.T @ X, d1m.T @ np.abs(X), t)
    within("gb1", grads.b1, d1.sum(0), d1m.sum(0), t)
    within("gW2", grads.W2, d2.T @ A, d2m.T @ A, t)
    within("gb2", grads.b2, d2.sum(0), d2m.sum(0), t)
    within("dX", dX, d1 @ W1, d1m @ np.abs(W1), h + k + 8)
    if mse:
        e = (Y - T) ** 2
        within("loss", loss, np.array([e.mean()]), np.array([e.mean()]), n * k + 4)


@pytest.mark.parametrize("n,din,dout,act", [(1, 1, 1, 0), (64, 64, 64, 1), (65, 65, 129, 0), (513, 40, 70, 1),
                                            (700, 300, 20, 0), (20000, 64, 256, 1)])
def test_dense_backward_edges(M, n, din, dout, act):
    from paper_1908_07847_amd._lib import lib
    say(f"dense backward n={n} {din}->{dout} act={act}")
    g = np.random.default_rng(n + dout)
    X = g.normal(size=(n, din)).astype(np.float32)
    Y = g.uniform(0.01, 0.99, (n, dout)).astype(np.float32)
    dY = g.normal(size=(n, dout)).astype(np.float32)
    W = g.uniform(-0.5, 0.5, (dout, din)).astype(np.float32)
    Xd, Yd, dYd, Wd = cuda(X), cuda(Y), cuda(dY), cuda(W)
    gW, gb, dX = torch.empty_like(Wd), torch.empty(dout, device="cuda"), torch.empty_like(Xd)
    ws = torch.empty(n * dout, device="cuda")      # the least the call accepts
    assert lib.mlp_dense_backward(Xd.data_ptr(), Yd.data_ptr(), dYd.data_ptr(), n, din, dout, Wd.data_ptr(), act,
                                  gW.data_ptr(), gb.data_ptr(), dX.data_ptr(), ws.data_ptr(), ws.numel() * 4, None) == 0
    torch.cuda.synchronize()
    X, Y, dY, W = (v.astype(np.float64) for v in (X, Y, dY, W))
    dZ = dY * (1 - Y * Y if act else Y * (1 - Y))
    mag = np.abs(dZ) + np.abs(dY) * Y              # 1 - Y Y and 1 - Y round to u of 1
    within("gW", gW, dZ.T @ X, mag.T @ np.abs(X), n + 6)
    within("gb", gb, dZ.sum(0), mag.sum(0), n + 6)
    within("dX", dX, dZ @ W, mag @ np.abs(W), dout + 6)


@pytest.mark.parametrize("n,din,dout,act", [(63, 64, 1, 0), (511, 65, 7, 1), (512, 48, 37, 0), (513, 129, 33, 1),
                                            (2048, 64, 195, 0), (2048, 63, 196, 1), (1562, 64, 256, 1),
                                            (1563, 64, 256, 0), (2049, 20, 3, 0)])
def test_dense_backward_few_rows(M, n, din, dout, act):   # both sides of the few-rows rule
    test_dense_backward_edges(M, n, din, dout, act)
