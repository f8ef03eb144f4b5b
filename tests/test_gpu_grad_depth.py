"""Depth of the float32 gradient sums: equal terms, whose roundings all go one
way, over more rows than one accumulator should take.

A range of rows is summed 16 from zero, those sums over at most 16,384 rows in
4 waves, and those in memory, then over the ranges: a parameter is
16 + min(r, 16384) / 64 + r / 16384 + ranges roundings deep (r rows a range), 2
where the waves meet, and its terms carry K + 8 of their own (u = 2^-24)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
U = 2.0 ** -24


def depth(n, ranges):
    r = -(-n // ranges)
    return 16 + min(r, 16384) / 64 + -(-r // 16384) + ranges + 2


def worst(got, value):
    return float((got.double() / value - 1.0).abs().max())


@pytest.mark.parametrize("n,d,h,k,net_rows,ranges", [
    (262144, 33, 64, 3, 64, 1),         # a workspace of one range
    (262144, 33, 64, 3, 262144, 512),   # ... and of all of them
    (40000, 20, 70, 5, 40000, 256),     # two unit tiles, more than four outputs
])
def test_backward_equal_terms(n, d, h, k, net_rows, ranges):
    from paper_1908_07847_amd import mlp
    print(f"backward n={n} {d}-{h}-{k}, workspace of {net_rows} rows", flush=True)
    x, a, y, up, w = (np.float32(v) for v in (0.7, 0.3, 0.6, 0.9, 0.35))
    net = mlp.Net(d, h, k, net_rows, theta=np.full(d * h + h + h * k + k, w, np.float32))
    full = lambda v, *s: torch.full(s, float(v), device="cuda")
    grads, _, _ = net.backward(full(x, n, d), full(a, n, h), full(y, n, k), dY=full(up, n, k))
    torch.cuda.synchronize()
    x, a, y, up, w = (float(v) for v in (x, a, y, up, w))
    d2 = up * y * (1 - y)
    d1 = k * d2 * w * a * (1 - a)
    bound = (depth(n, ranges) + k + 8) * U
    for name, got, value in (("gW1", grads.W1, n * d1 * x), ("gb1", grads.b1, n * d1), ("gW2", grads.W2, n * d2 * a),
                             ("gb2", grads.b2, n * d2)):
        assert worst(got, value) <= bound, (name, worst(got, value), bound)


@pytest.mark.parametrize("n,din,dout,ranges", [(40000, 1024, 2048, 1),    # 512 tiles: one range
                                               (100000, 1024, 512, 4)])
def test_dense_equal_terms(n, din, dout, ranges):
    from paper_1908_07847_amd._lib import lib
    print(f"dense n={n} {din}->{dout}", flush=True)
    x, y, up = (np.float32(v) for v in (0.7, 0.6, 0.9))
    full = lambda v, *s: torch.full(s, float(v), device="cuda")
    X, Y, dY, W = full(x, n, din), full(y, n, dout), full(up, n, dout), full(0.1, dout, din)
    gW, gb, ws = torch.empty_like(W), torch.empty(dout, device="cuda"), torch.empty(n * dout, device="cuda")
    assert lib.mlp_dense_backward(X.data_ptr(), Y.data_ptr(), dY.data_ptr(), n, din, dout, W.data_ptr(), 0,
                                  gW.data_ptr(), gb.data_ptr(), None, ws.data_ptr(), ws.numel() * 4, None) == 0
    torch.cuda.synchronize()
    x, y, up = (float(v) for v in (x, y, up))
    dz = up * y * (1 - y)
    bound = (depth(n, ranges) + 8) * U
    assert worst(gW, n * dz * x) <= bound, (worst(gW, n * dz * x), bound)
    assert worst(gb, n * dz) <= bound, (worst(gb, n * dz), bound)
