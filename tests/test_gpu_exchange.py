"""The large-N trainer's exchanges: the W1 copy the update writes (float32,
padded rows), the partial gradients' tile order and the split of their sums,
at sizes where rows, tiles and quads are ragged."""
import sys

import numpy as np
import pytest
import torch

import oracle
from oracle import Params
from paper_1908_07847_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    from paper_1908_07847_amd import mlp
    return mlp


def problem(n, d, h, k, seed):
    g = np.random.default_rng(seed)
    X = g.standard_normal((n, d)).astype(np.float32)
    T = np.zeros((n, k), np.float32)
    T[np.arange(n), g.integers(0, k, n)] = 1.0
    return X, T, g.uniform(-0.5, 0.5, d * h + h + h * k + k).astype(np.float32)


@pytest.mark.parametrize("d,h,batch", [(64, 1024, 4096), (33, 256, 4096), (7, 100, 512), (1, 64, 128)])
def test_w1_copy_equals_staging_from_theta(M, d, h, batch):
    """After a launch's first step W1 is staged from the copy the update wrote:
    one launch of three one-step epochs equals three launches, bitwise."""
    print(f"float32 W1 copy: {d}-{h}-3, {batch} rows", flush=True)
    sys.stdout.flush()
    X, T, th = problem(batch, d, h, 3, d + h)
    Xd, Td = torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda()
    a = M.Net(d, h, 3, 2 * batch, batch=batch, theta=th)   # (minibatch shape: the large-N trainer)
    X2, T2 = torch.cat([Xd, Xd]), torch.cat([Td, Td])
    a.train(X2, T2, 3)
    b = M.Net(d, h, 3, batch, batch=batch, theta=th)
    for _ in range(6):                                       # the same rows, one step a launch
        b.train(Xd, Td, 1)
    torch.cuda.synchronize()
    if h > 64 or batch > 128:                                # (the smallest shape trains b full batch in one workgroup)
        assert torch.equal(a.flat, b.flat) and torch.equal(a.comp, b.comp)
    else:
        assert float((a.flat - b.flat).abs().max()) <= 1e-6


@pytest.mark.parametrize("n,d,h,k,batch,grid", [
    (1000, 17, 65, 3, 256, None),      # one unit in a second tile block, short last minibatch
    (4096, 48, 256, 4, 1024, (32, 4)),  # exactly three feature blocks, four outputs
    (2048, 49, 300, 1, 2048, None),    # one feature in the fourth block, full batch
    (640, 64, 64, 2, 64, (2, 1)),      # few row blocks: the sums split over threads, not rows
])
def test_partial_order_matches_the_oracle(M, n, d, h, k, batch, grid):
    print(f"partials: {n} rows {d}-{h}-{k} batch {batch} grid {grid}", flush=True)
    X, T, th = problem(n, d, h, k, n + d)
    if grid:
        M.set_launch_hint(large_grid=grid)
    try:
        net = M.Net(d, h, k, n, batch=batch, theta=th)
        hist = net.train(torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda(), 2)
        torch.cuda.synchronize()
    finally:
        M.reset_launch_hint()
    q, ref = oracle.train(X, T, Params.of(synth.Theta.unpack(th, d, h, k)), 0.1, 2, batch=batch)
    got = synth.Theta.unpack(net.flat.cpu().numpy(), d, h, k)
    for a, b in ((got.W1, q.W1), (got.b1, q.b1), (got.W2, q.W2), (got.b2, q.b2), (hist.cpu().numpy(), ref)):
        assert np.max(np.abs(a - b)) <= 1e-5 * np.max(np.abs(b))   # the trainers' stated tolerance
