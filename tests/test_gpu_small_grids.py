"""Minibatches of few rows: grids of few workgroups, whose update gives a thread
parameters and not quads of the partial order, against the FP64 oracle and
against the other order (8 waves), which adds the same partials alike."""
import numpy as np
import pytest
import torch

import oracle
from oracle import Params
from paper_1908_07847_amd import synth
from test_gpu_exchange import M, problem   # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,h,k,batch", [
    (200, 33, 4, 3, 32),      # one workgroup, fewer parameters than threads; a short last minibatch
    (330, 64, 64, 4, 32),     # more than one batch of parameters a thread
    (300, 1, 70, 1, 96),      # one feature, one output, two workgroups
    (640, 64, 300, 2, 160),   # five hidden blocks
    (768, 17, 1000, 3, 96),   # sixteen, one row block
    (1024, 48, 600, 3, 64),   # two row blocks
])
def test_small_grids_match_the_oracle(M, n, d, h, k, batch):   # noqa: F811
    print(f"small grid: {n} rows {d}-{h}-{k} batch {batch}", flush=True)
    X, T, th = problem(n, d, h, k, n + d)
    net = M.Net(d, h, k, n, batch=batch, theta=th)
    hist = net.train(torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda(), 2)
    torch.cuda.synchronize()
    q, ref = oracle.train(X, T, Params.of(synth.Theta.unpack(th, d, h, k)), 0.1, 2, batch=batch)
    got = synth.Theta.unpack(net.flat.cpu().numpy(), d, h, k)
    for a, b in ((got.W1, q.W1), (got.b1, q.b1), (got.W2, q.W2), (got.b2, q.b2), (hist.cpu().numpy(), ref)):
        assert np.max(np.abs(a - b)) <= 1e-5 * np.max(np.abs(b))   # the trainers' stated tolerance


@pytest.mark.parametrize("prec", ["fp32", "bf16", "e4m3"])
@pytest.mark.parametrize("compensated", [True, False])
@pytest.mark.parametrize("d,h,k,batch,grid", [(33, 4, 3, 32, (1, 1)), (64, 64, 4, 32, (1, 1)), (1, 130, 1, 64, (2, 4)),
                                              (40, 200, 2, 160, (1, 4))])
def test_update_orders_agree(M, d, h, k, batch, grid, prec, compensated):   # noqa: F811
    """Bitwise: 4 waves update by parameters, 8 by quads, each adding a
    parameter's row blocks in order."""
    n = 5 * batch - 7
    print(f"update orders: {n} rows {d}-{h}-{k} batch {batch} {prec} compensated={compensated}", flush=True)
    X, T, th = problem(n, d, h, k, d + h)
    Xd, Td = torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda()
    nets = []
    try:
        for waves in (4, 8):
            M.set_launch_hint(large_grid=grid, large_waves=waves)
            net = M.Net(d, h, k, n, batch=batch, theta=th, prec=prec, compensated=compensated)
            hist = net.train(Xd, Td, 3)
            torch.cuda.synchronize()
            nets.append((net, hist.cpu().numpy()))
    finally:
        M.reset_launch_hint()
    (a, ha), (b, hb) = nets
    assert torch.equal(a.flat, b.flat)
    if compensated:
        assert torch.equal(a.comp, b.comp)
    assert np.max(np.abs(ha - hb)) <= 1e-6 * np.max(np.abs(hb))   # the losses' waves add in another order
