"""Depth of the trainers' gradient sums.  All 128 rows of a network are the same
row, so every term of a gradient is the same number; a network of that one row
has the sum as its gradient (2 / (n K) scales by a power of two).  At learning
rate 1e6 the parameters after one epoch show the gradients.

A chain of m equal terms, one rounding per step, is off by at most m / 2
roundings of its result (step k rounds k terms); adding q such sums by at most
q / 2 + 1 more.  The reference, the scaling by the rate and the subtraction
add 5 (u = 2^-24)."""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
U, LR, N = 2.0 ** -24, 1e6, 128


def check(th, many, one, chain, sums):
    """many, one: parameters after the epoch on 128 rows and on one."""
    th, gm, g1 = th.astype(np.float64), th - many.astype(np.float64), th - one.astype(np.float64)
    on = np.abs(g1) > 50 * np.abs(th)     # the parameters are mostly gradient
    assert on.mean() > 0.5
    worst = float(np.max(np.abs(gm[on] / g1[on] - 1.0))) / U
    assert worst <= chain / 2 + sums / 2 + 1 + 5, worst


@pytest.mark.parametrize("nets,d,h,chain,sums", [
    (300, 33, 33, 32, 4),    # above one net per CU, over 32 units: a wave per 16 units, all rows, two tiles a chain
    (300, 48, 64, 32, 4),
    (300, 33, 32, 32, 4),    # up to 32 units: 4 waves split the rows
    (40, 48, 64, 16, 8),     # up to one net per CU: 8 waves split the rows
])
def test_batched_equal_rows(nets, d, h, chain, sums):
    from paper_1908_07847_amd import mlp
    print(f"batched {nets} nets {d}-{h}-3", flush=True)
    g = np.random.default_rng(h)
    P = d * h + h + 3 * h + 3
    x = g.normal(size=(nets, 1, d)).astype(np.float32)
    t = g.random((nets, 1, 3)).astype(np.float32)
    th = g.uniform(-0.5, 0.5, (nets, P)).astype(np.float32)
    after = []
    for n in (N, 1):
        plan = mlp.BatchPlan([dict(n_rows=n, n_hidden=h, lr=LR, x_off=i * n, p_off=i * P) for i in range(nets)])
        theta = torch.from_numpy(th.reshape(-1)).cuda()
        mlp.train_batched(plan, torch.from_numpy(np.repeat(x, n, 1).reshape(-1, d)).cuda(),
                          torch.from_numpy(np.repeat(t, n, 1).reshape(-1, 3)).cuda(), theta, None, 1, d, 3)
        torch.cuda.synchronize()
        after.append(theta.cpu().numpy().reshape(nets, P)[:, :d * h + h])
    check(th[:, :d * h + h], *after, chain, sums)


@pytest.mark.parametrize("widths", [(33, 16, 3), (33, 16, 16, 3), (10, 8, 8, 8, 2), (33, 60, 3)])
def test_deep_equal_rows(widths):
    from paper_1908_07847_amd._lib import lib
    print(f"deep {widths}", flush=True)
    P = sum(a * b + b for a, b in zip(widths, widths[1:]))
    nw = widths[0] * widths[1]
    w = (ctypes.c_int32 * len(widths))(*widths)
    ths, many, one = [], [], []
    for seed in range(100):
        g = np.random.default_rng(seed)
        x = g.normal(size=(1, widths[0])).astype(np.float32)
        t = g.random((1, widths[-1])).astype(np.float32)
        th = g.uniform(-0.5, 0.5, P).astype(np.float32)
        for n, out in ((N, many), (1, one)):
            X, T = (torch.from_numpy(np.repeat(v, n, 0)).cuda() for v in (x, t))
            theta = torch.from_numpy(th).cuda()
            assert lib.mlp_deep_train(X.data_ptr(), T.data_ptr(), n, len(widths) - 1, w, 0, theta.data_ptr(), None, LR,
                                      1, None, None) == 0
            torch.cuda.synchronize()
            out.append(theta.cpu().numpy()[:nw])
        ths.append(th[:nw])
    check(np.stack(ths), np.stack(many), np.stack(one), 16, 8)
