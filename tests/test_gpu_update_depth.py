"""The large-N trainer's sum of partial gradients over the row blocks.

A switch unit saturates the outputs of a row, whose deltas are then exactly
zero; so with one open row in every row block the partial gradients are one
row's, and a step's gradient is their sum up to the roundings of that sum
alone.  The terms are read from steps with a single open row, and all of them
exactly, from the compensated update at rate 1.

Bound: rows of different data, so the roundings are independent; an add that
returns s rounds by up to ulp(s) / 2, uniformly, at most u |s| / sqrt(3) rms,
u = 2^-24.  The sum has to be no worse than four chains of consecutive row
blocks that meet in a tree."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
U = 2.0 ** -24


@pytest.fixture(scope="module")
def M():
    from paper_1908_07847_amd import mlp
    return mlp


def gradient(M, X, T, theta, shape, b):
    d, h, k = shape
    net = M.Net(d, h, k, b, batch=b, lr=1.0, theta=theta)
    net.train(X, T, 1)
    torch.cuda.synchronize()
    new, c = net.flat.cpu().numpy().astype(np.float64), net.comp.cpu().numpy().astype(np.float64)
    return c - (new - theta.astype(np.float64))      # -y of t = w + y, c = (t - w) - y


@pytest.mark.parametrize("b,d,h,blocks", [
    (4096, 33, 256, 64), (16384, 33, 64, 256),
    (8192, 48, 512, 64),        # 8 waves
])
def test_sum_over_row_blocks(M, b, d, h, blocks):
    print(f"row blocks' sum b={b} {d}-{h}-3", flush=True)
    k, per = 3, b // blocks
    plan = M.large_plan(d, h, k, b, batch=b, n_cu=256)
    assert plan["row_blocks"] == blocks and plan["row_blocks"] * plan["hidden_blocks"] == 256
    g = np.random.default_rng(h)
    W1, b1 = g.uniform(0.1, 0.5, (h, d)), g.uniform(0.1, 0.5, h)
    W2, b2 = g.uniform(0.1, 0.5, (k, h)) * np.where(np.arange(h) % 2, 1, -1), g.uniform(0.1, 0.5, k)
    W1[0] = 0.1
    W1[0, 0], b1[0], W2[:, 0] = 300.0, -200.0, 300.0
    theta = np.concatenate([v.ravel() for v in (W1, b1, W2, b2)]).astype(np.float32)
    x = g.uniform(0.1, 1.0, (blocks, d)).astype(np.float32)
    x[:, 0] = 0.0
    shut = x[0].copy()
    shut[0] = 1.0
    T = torch.zeros(b, k, device="cuda")
    opened = torch.from_numpy(x).cuda()

    def with_open(which):
        X = torch.from_numpy(shut).cuda().repeat(b, 1)
        X[np.array(which) * per] = opened[which]
        return gradient(M, X, T, theta, (d, h, k), b)

    terms = np.stack([with_open([i]) for i in range(blocks)])
    total = with_open(list(range(blocks)))
    on = np.all(np.abs(terms) > 1e-12, axis=0)
    assert np.sum(on) > 0.9 * theta.size
    assert np.all(np.abs(total[on]) < 0.1)            # smaller than the parameters: the compensation is exact
    terms = terms[:, on]
    exact = terms.sum(0)
    chains = [terms[blocks * i // 4:blocks * (i + 1) // 4].cumsum(0) for i in range(4)]
    ends = [v[-1] for v in chains]
    adds = [v[1:] for v in chains] + [np.array([ends[0] + ends[1], ends[2] + ends[3], exact])]
    sq = sum((v ** 2).sum(0) for v in adds) * U ** 2 / 3
    rms = float(np.sqrt(np.mean(sq / exact ** 2)))
    got = float(np.sqrt(np.mean((total[on] / exact - 1.0) ** 2)))
    print(f"rms {got / U:.3f} u, bound {rms / U:.3f} u")
    assert got <= rms
