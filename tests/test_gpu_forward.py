"""The forward / prediction kernel for up to 64 inputs and 4 outputs at the
edges of its tiles (16 units, 4 features, 32 rows per wave, 256-unit blocks),
against float64, and its classes and count against its own outputs."""
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


@pytest.mark.parametrize("n,d,h,k,act", [
    (1, 1, 1, 1, "sigmoid"),        # one of everything
    (33, 4, 17, 2, "tanh"),         # one past a wave's rows and a unit tile
    (128, 64, 256, 4, "sigmoid"),   # the largest contraction, one whole block
    (129, 33, 257, 3, "sigmoid"),   # one unit in a second block
    (1000, 61, 600, 3, "tanh"),     # three blocks, ragged everywhere
    (200000, 33, 16, 3, "sigmoid"), # several rounds of the resident grid
])
def test_forward_and_predict_edges(M, n, d, h, k, act):
    print(f"forward n={n} {d}-{h}-{k} {act}", flush=True)
    sys.stdout.flush()
    g = np.random.default_rng(n + d)
    X = g.normal(size=(n, d)).astype(np.float32)
    T = np.zeros((n, k), np.float32)
    T[np.arange(n), g.integers(0, k, n)] = g.integers(0, 2, n) if k == 1 else 1.0
    theta = g.uniform(-0.5, 0.5, d * h + h + h * k + k).astype(np.float32)
    net = M.Net(d, h, k, min(n, 4096), batch=min(n, 4096), theta=theta, act=act)
    Xd, Td = torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda()
    A, Y = net.forward(Xd)
    Y2, labels, correct = net.predict(Xd, Td)
    torch.cuda.synchronize()
    W1, b1 = theta[:d * h].reshape(h, d).astype(np.float64), theta[d * h:d * h + h].astype(np.float64)
    W2 = theta[d * h + h:d * h + h + k * h].reshape(k, h).astype(np.float64)
    z1 = X.astype(np.float64) @ W1.T + b1
    Ar = np.tanh(z1) if act == "tanh" else 1 / (1 + np.exp(-z1))
    z2 = Ar @ W2.T + theta[-k:].astype(np.float64)
    # z1: d + 1 roundings of its sum of |terms|; the activations have slope at
    # most 1 and a few ulps of their own; z2 the same over h + 1 terms, sigma' <= 1/4
    e1 = (d + 2) * U * (np.abs(X) @ np.abs(W1).T + np.abs(b1)) + 4 * U
    e2 = e1 @ np.abs(W2).T + (h + 2) * U * (np.abs(Ar) @ np.abs(W2).T + 0.5)
    assert np.all(np.abs(A.cpu().numpy() - Ar) <= e1)
    Yh = Y.cpu().numpy()
    assert np.all(np.abs(Yh - 1 / (1 + np.exp(-z2))) <= 0.25 * e2 + 4 * U)
    assert torch.equal(Y, Y2)
    cls = lambda v: (v[:, 0] > 0.5).astype(np.int32) if k == 1 else v.argmax(1).astype(np.int32)
    assert np.array_equal(labels.cpu().numpy(), cls(Yh))
    assert int(correct) == int((cls(Yh) == cls(T)).sum())
    assert torch.equal(net.predict(Xd)[1], labels)     # without targets
