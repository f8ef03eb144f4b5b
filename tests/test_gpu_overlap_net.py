"""mlp_backward with outputs over Y, dY or T.  dX (as many outputs as inputs):
the bits of the call with separate memory.  Gradients and the loss: on small
dyadic numbers, whose products and sums are exact in float32 in any order,
float64's results."""
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


@pytest.mark.parametrize("over", ["Y", "dY", "T"])
@pytest.mark.parametrize("n,d,h,k", [
    (64, 3, 2, 4),              # a workgroup per unit
    (2048, 20, 300, 2),         # one range of rows and several
    (4096, 33, 20, 4), (16384, 70, 16, 8),
])
def test_gradients_over_inputs(n, d, h, k, over):
    from paper_1908_07847_amd import mlp as M
    from paper_1908_07847_amd._lib import lib, Params
    mse = over == "T"
    print(f"backward gradients over {over}: n={n} {d}-{h}-{k}", flush=True)
    g = np.random.default_rng(n)
    pick = lambda v, *shape: g.choice(np.array(v, np.float64), shape)
    X, W2, A = pick([-2, -1, 1, 2], n, d), pick([-1, 1], k, h), pick([0, 0.5], n, h)
    Y, T, dY = np.full((n, k), 0.5), pick([0, 1, 1.5], n, k), pick([-1, 1], n, k)
    theta = np.concatenate([np.ones(d * h), np.zeros(h), W2.ravel(), np.zeros(k)]).astype(np.float32)
    net = M.Net(d, h, k, n, theta=theta)
    dev = {a: torch.from_numpy(v.astype(np.float32)).cuda() for a, v in
           dict(X=X, A=A, Y=Y, T=T, dY=dY).items()}
    flat, out = dev[over].view(-1), {}
    at = 1                                     # the loss, then the gradients that fit
    for name, shape in (("b1", (h,)), ("b2", (k,)), ("W2", (k, h)), ("W1", (h, d))):
        size = int(np.prod(shape))
        if at + size <= flat.numel():
            out[name], at = flat[at:at + size].view(shape), at + size
        else:
            out[name] = torch.empty(shape, device="cuda")
    grads = Params(*(out[a].data_ptr() for a in ("W1", "b1", "W2", "b2")))
    assert lib.mlp_backward(net._h, *(dev[a].data_ptr() for a in ("X", "A", "Y")), None if mse else dev["dY"].data_ptr(),
                            dev["T"].data_ptr(), n, grads, None, flat.data_ptr() if mse else None, None) == 0
    torch.cuda.synchronize()
    scale = 2.0 / (n * k) if mse else 1.0      # a power of two
    d2 = (scale * (Y - T) if mse else dY) * 0.25
    d1 = (d2 @ W2) * A * (1 - A)
    assert np.max(np.abs(d1).T @ np.abs(X)) < 2 ** 24 * scale / 32
    for name, ref in dict(W1=d1.T @ X, b1=d1.sum(0), W2=d2.T @ A, b2=d2.sum(0)).items():
        assert np.array_equal(out[name].cpu().numpy(), ref), name
    if mse:
        assert float(flat[0]) == np.mean((Y - T) ** 2)
