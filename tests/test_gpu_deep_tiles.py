"""One-launch training of several hidden layers on the matrix cores, at the
edges of its 16-row and 16-unit tiles and of the shapes it takes (wider layers
and larger nets go to the lane-per-entry form), against the FP64 oracle."""
import sys

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    from paper_1908_07847_amd import mlp
    return mlp


@pytest.mark.parametrize("widths,rows,act,epochs", [
    ([5, 16, 16, 3], 16, "sigmoid", 200),        # one row tile, whole unit tiles
    ([33, 17, 15, 4], 17, "tanh", 200),          # one row and one unit past a tile
    ([70, 32, 3], 120, "sigmoid", 100),          # five input tiles
    ([16, 64, 49, 20], 33, "tanh", 100),         # four unit tiles, twenty outputs
    ([8, 8, 8, 3], 300, "sigmoid", 100),         # nineteen row tiles on sixteen waves
    ([12, 65, 3], 40, "sigmoid", 100),           # a layer of 65 units: the other form
])
def test_tiled_deep_training_matches_the_oracle(M, widths, rows, act, epochs):
    print(f"deep tiles {widths} on {rows} rows, {act}, {epochs} epochs", flush=True)
    sys.stdout.flush()
    g = np.random.default_rng(rows)
    X = g.normal(size=(rows, widths[0])).astype(np.float32)
    T = np.zeros((rows, widths[-1]), np.float32)
    T[np.arange(rows), g.integers(0, widths[-1], rows)] = 1.0
    theta = g.uniform(-0.5, 0.5, oracle.deep_n_params(widths)).astype(np.float32)
    net = M.DeepNet(widths, theta=theta, act=act)
    hist = net.train_kernel(torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda(), epochs)
    torch.cuda.synchronize()
    q, ref = oracle.deep_train(X, T, widths, theta, 0.1, epochs, act=act)
    got = net.flat.detach().cpu().numpy()
    assert np.max(np.abs(got - q)) <= 1e-5 * np.max(np.abs(q))     # the trainers' stated tolerance
    assert np.max(np.abs(hist.cpu().numpy() - ref)) <= 1e-5 * np.max(np.abs(ref))
