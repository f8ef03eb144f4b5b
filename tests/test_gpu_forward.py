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


@pytest.mark.parametrize("d,k", [(1, 1), (33, 3), (64, 4), (70, 2)])   # 70 inputs: the general kernel
def test_eval_edges(M, d, k):
    """Networks of 1 .. 300 units on 1 .. 200 rows (one past a wave's tiles and
    a round's rows) in one evaluation, against float64."""
    shapes = [(1, 1), (32, 16), (33, 17), (25, 64), (200, 65), (7, 300)]
    print(f"eval d={d} k={k} {shapes}", flush=True)
    g = np.random.default_rng(d)
    items, xs, ts, th, row, off, ref = [], [], [], [], 0, 0, []
    for n, h in shapes:
        X = g.normal(size=(n, d)).astype(np.float32)
        T = np.zeros((n, k), np.float32)
        T[np.arange(n), g.integers(0, k, n)] = g.integers(0, 2, n) if k == 1 else 1.0
        p = g.uniform(-0.5, 0.5, d * h + h + h * k + k).astype(np.float32)
        items.append(dict(n_rows=n, n_hidden=h, lr=0.0, x_off=row, p_off=off))
        W1, b1 = p[:d * h].reshape(h, d).astype(np.float64), p[d * h:d * h + h].astype(np.float64)
        A = 1 / (1 + np.exp(-(X.astype(np.float64) @ W1.T + b1)))
        Y = 1 / (1 + np.exp(-(A @ p[d * h + h:-k].reshape(k, h).T.astype(np.float64) + p[-k:])))
        cls = lambda v: (v[:, 0] > 0.5) if k == 1 else v.argmax(1)
        srt = np.sort(Y, 1)
        near = int(((np.abs(Y[:, 0] - 0.5) if k == 1 else srt[:, -1] - srt[:, -2]) < 1e-5).sum())
        ref.append((np.mean((Y - T) ** 2), int((cls(Y) == cls(T)).sum()), near))
        xs.append(X), ts.append(T), th.append(p)
        row, off = row + n, off + p.size
    plan = M.BatchPlan(items)
    cat = lambda v: torch.from_numpy(np.concatenate(v)).cuda()
    loss, correct = M.eval_batched(plan, cat(xs), cat(ts), cat(th), d, k)
    torch.cuda.synchronize()
    for i, (l, c, near) in enumerate(ref):
        # an output is within (d + h + 8) u of its sums' size, below 1e-5 here
        assert abs(float(loss[i]) - l) <= 2e-5 * l + 1e-9, (i, float(loss[i]), l)
        assert abs(int(correct[i]) - c) <= near, (i, int(correct[i]), c)


@pytest.mark.parametrize("n,ng", [(1, 1), (513, 64), (3000, 4096), (9001, 4097), (5000, 65536)])
def test_cv_select_group_waves(M, n, ng):
    """One group per wave up to 4096 groups, several above: every mean is the
    float32 sum in increasing net order, so the comparison is exact."""
    print(f"cv_select n={n} groups={ng}", flush=True)
    g = np.random.default_rng(n)
    loss = g.uniform(0.1, 1, n).astype(np.float32)
    grp = g.integers(-1, ng + 1, n).astype(np.int32)      # some belong to no group
    s, c = np.zeros(ng, np.float32), np.zeros(ng, np.int64)
    for l, q in zip(loss, grp):
        if 0 <= q < ng:
            s[q] = np.float32(s[q] + l)
            c[q] += 1
    with np.errstate(divide="ignore", invalid="ignore"):
        want = np.where(c > 0, s / c.astype(np.float32), np.float32(np.inf)).astype(np.float32)
    mean, best = M.cv_select(torch.from_numpy(loss).cuda(), torch.from_numpy(grp).cuda(), ng)
    torch.cuda.synchronize()
    assert np.array_equal(mean.cpu().numpy(), want)
    assert int(best) == int(np.argmin(want))
