"""A workspace of the queried size covers every grid that a launch hint may ask
for: 961 units in 15 hidden blocks are padded to 1920, more than in 16 or 8."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid", [(17, 15), (16, 16), (32, 8)])
def test_hint_grid_fits_the_queried_workspace(grid):
    from paper_1908_07847_amd import mlp
    n, d, h, k = 17 * 32 * 512, 64, 961, 1
    print(f"{n} rows, {d}-{h}-{k} on {grid}", flush=True)
    g = np.random.default_rng(5)
    X = torch.from_numpy(g.normal(size=(n, d)).astype(np.float32)).cuda()
    T = torch.from_numpy(g.random((n, k)).astype(np.float32)).cuda()
    theta = g.uniform(-0.1, 0.1, d * h + h + h * k + k).astype(np.float32)
    out = []
    for hint in (None, grid):
        net = mlp.Net(d, h, k, n, theta=theta, lr=0.5)
        try:
            if hint:
                mlp.set_launch_hint(large_grid=hint)
            net.train(X, T, 1)
            torch.cuda.synchronize()
        finally:
            mlp.reset_launch_hint()
        out.append(net.flat.cpu().numpy().astype(np.float64))
    step = np.abs(out[0] - theta).max()
    # the same gradient in another summation order: n + h + d roundings at most
    assert np.abs(out[0] - out[1]).max() <= (n + h + d) * 2.0 ** -24 * step + 1e-7
