"""mlp_backward with dX over Y, dY or T (as many outputs as inputs): the bits
of the call with separate memory."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("over", ["Y", "dY", "T"])
@pytest.mark.parametrize("n,d,h", [(1, 1, 1), (65, 3, 70), (513, 4, 20), (3000, 16, 130)])
def test_backward_overlaps(n, d, h, over):
    from paper_1908_07847_amd import mlp as M
    from paper_1908_07847_amd._lib import lib
    print(f"backward dX over {over}: n={n} {d}-{h}-{d}", flush=True)
    g = np.random.default_rng(n)
    X, A, Y, T = (torch.from_numpy(g.uniform(0.01, 0.99, (n, w)).astype(np.float32)).cuda() for w in (d, h, d, d))
    net = M.Net(d, h, d, n, theta=g.uniform(-0.5, 0.5, 2 * d * h + h + d).astype(np.float32))
    mse = over == "T"
    up = None if mse else T
    ref, dX, _ = net.backward(X, A, Y, dY=up, T=T if mse else None, want_dx=True)
    mem = {"Y": Y.clone(), "dY": T.clone(), "T": T.clone()}
    got = net.new_grads()
    ptr = lambda k: mem[k].data_ptr()
    loss = torch.empty(4, device="cuda")
    assert lib.mlp_backward(net._h, X.data_ptr(), A.data_ptr(), ptr("Y"), None if mse else ptr("dY"),
                            ptr("T") if mse else None, n, got.c(), ptr(over), loss.data_ptr(), None) == 0
    torch.cuda.synchronize()
    assert torch.equal(mem[over], dX)
    for a, b in zip((got.W1, got.b1, got.W2, got.b2), (ref.W1, ref.b1, ref.W2, ref.b2)):
        assert torch.equal(a, b)
