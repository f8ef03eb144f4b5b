"""mlp_predict and mlp_cv_select with outputs over inputs: the bits of the
calls with separate memory."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    from paper_1908_07847_amd import mlp
    return mlp


@pytest.mark.parametrize("n,d,h,k,out,over", [
    (1, 1, 1, 1, "labels", "X"), (700, 33, 10, 3, "labels", "X"), (5000, 5, 300, 4, "correct", "X"),
    (700, 3, 10, 1, "labels", "Y"), (100, 33, 16, 3, "labels", "theta"),
    (3000, 40, 64, 2, "correct", "theta"),
])
def test_predict(M, n, d, h, k, out, over):
    from paper_1908_07847_amd._lib import lib
    print(f"predict {out} over {over}: n={n} {d}-{h}-{k}", flush=True)
    g = np.random.default_rng(n)
    theta = g.uniform(-0.5, 0.5, d * h + h + h * k + k).astype(np.float32)
    X = torch.from_numpy(g.normal(size=(n, d)).astype(np.float32)).cuda()
    T = torch.from_numpy((g.random((n, k)) < 0.4).astype(np.float32)).cuda()
    net = M.Net(d, h, k, n, theta=theta)
    Y, labels, correct = net.predict(X, T)
    mem = dict(X=X.clone(), T=T.clone(), Y=torch.empty_like(Y), theta=net.flat)
    outs = dict(labels=torch.empty(max(n, 4), dtype=torch.int32, device="cuda")[:n],
                correct=torch.empty(4, dtype=torch.int32, device="cuda")[:1])
    outs[out] = mem[over].view(-1).view(torch.int32)[:n if out == "labels" else 1]
    assert outs[out].numel() == (n if out == "labels" else 1)
    assert lib.mlp_predict(net._h, mem["X"].data_ptr(), n, mem["Y"].data_ptr(), outs["labels"].data_ptr(),
                           mem["T"].data_ptr(), outs["correct"].data_ptr(), None) == 0
    torch.cuda.synchronize()
    assert torch.equal(outs["labels"], labels) and torch.equal(outs["correct"], correct)
    if over != "Y":
        assert torch.equal(mem["Y"], Y)


@pytest.mark.parametrize("over", ["loss", "group"])
@pytest.mark.parametrize("n,groups", [(1, 1), (64, 17), (128, 128), (129, 100), (1024, 1024), (5000, 1000)])
def test_cv_select(M, n, groups, over):
    from paper_1908_07847_amd._lib import lib
    print(f"cv_select means over {over}: {n} nets in {groups} groups", flush=True)
    g = np.random.default_rng(n)
    loss = torch.from_numpy(g.random(n).astype(np.float32)).cuda()
    group = torch.from_numpy(g.integers(-1, groups + 1, n).astype(np.int32)).cuda()
    mean, best = (torch.empty(max(groups, 4), device="cuda")[:groups], torch.empty(4, dtype=torch.int32, device="cuda")[:1])
    call = lambda l, q, m, b: lib.mlp_cv_select(l.data_ptr(), q.data_ptr(), n, groups, m.data_ptr(), b.data_ptr(), None)
    assert call(loss, group, mean, best) == 0
    mem = dict(loss=loss.clone(), group=group.clone())
    over_mean = mem[over].view(torch.float32)[:groups]
    b2 = torch.empty_like(best)
    assert call(mem["loss"], mem["group"], over_mean, b2) == 0
    torch.cuda.synchronize()
    assert torch.equal(over_mean, mean) and torch.equal(b2, best)
