"""What is timed: the calls that a user of this package makes, over the range
of sizes they are made at.

Each case is one call path through the package's public entry points:

  small     Net.train, full batch, all epochs in one launch (the paper's own
            kind of network: tens of rows, tens of hidden units)
  autograd  MLPFunction forward, torch's MSE, the adjoint, Net.step
  batched   train_batched over many small networks (cross-validation grid)
  readout   eval_batched on the held-out folds, then cv_select
  minibatch Net.train on a large table in minibatches (fp32, bf16, e4m3)
  shared    train_shared: several networks on one table (learning-rate grid)
  predict   Net.predict on a large table, with targets
  deep      DeepNet.train_kernel: several hidden layers, one launch
  layers    DeepNet.train_fused: several hidden layers at sizes beyond one
            workgroup, one library call per layer

Inputs have the distributions of the package's generator: z-scored Gaussian
and Bernoulli columns, one-hot classes of a random teacher network, initial
parameters from U(-0.5, 0.5).
"""
from __future__ import annotations

import math

import torch

from paper_1908_07847_amd import mlp

LR = 0.1


def listed():
    return [
        # the smallest call: the paper's network on 60 patients, latency alone
        dict(name="small_60x33_h10", kind="small", n=60, d=33, h=10, k=3, epochs=1000, act="sigmoid", mu=0.0),
        # one differentiable step of a small network inside a torch program
        dict(name="autograd_120x33_h16", kind="autograd", n=120, d=33, h=16, k=3, act="sigmoid", dx=False),
        # the same inside a program with a large table, ragged in its rows
        dict(name="autograd_50000x33_h256", kind="autograd", n=50000, d=33, h=256, k=3, act="sigmoid", dx=False),
        # a hyperparameter grid with five folds: 4096 networks at once
        dict(name="batched_4096", kind="batched", nets=4096, d=33, k=3, h_max=64, epochs=100),
        # choosing among them: held-out losses and the best group
        dict(name="readout_4096", kind="readout", nets=4096, d=33, k=3, h_max=64),
        # a large table in minibatches, moderate network, one epoch
        dict(name="minibatch_1048576x33_h256", kind="minibatch", n=1 << 20, d=33, h=256, k=3, batch=4096,
             prec="fp32", epochs=1),
        # the largest: the wide network on 4 M rows, one epoch
        dict(name="minibatch_4194304x64_h1024", kind="minibatch", n=1 << 22, d=64, h=1024, k=3, batch=16384,
             prec="fp32", epochs=1),
        # the wide network with 8-bit operands, part of an epoch
        dict(name="minibatch_524288x64_h1024_e4m3", kind="minibatch", n=1 << 19, d=64, h=1024, k=3, batch=16384,
             prec="e4m3", epochs=1),
        # a grid of learning rates and initialisations on one table, bf16
        dict(name="shared_64_131072x64_h1024_bf16", kind="shared", nets=64, n=1 << 17, d=64, h=1024, k=3,
             batch=16384, prec="bf16", epochs=1),
        # classifying a large table
        dict(name="predict_1048576x33_h256", kind="predict", n=1 << 20, d=33, h=256, k=3, act="sigmoid"),
        # two hidden layers on 120 patients, every epoch in one launch
        dict(name="deep_120_33_16_16_3", kind="deep", n=120, d=33, h=16, h2=16, k=3, act="sigmoid", epochs=500),
        # two hidden layers on a table that no single workgroup holds
        dict(name="layers_20000_64_256_64_3", kind="layers", n=20000, d=64, h=256, h2=64, k=3, act="tanh", epochs=2),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges."""
    kind = rng.choice(["small", "autograd", "autograd", "batched", "readout", "minibatch", "minibatch", "minibatch",
                       "shared", "predict", "deep", "layers"])
    act = rng.choice(["sigmoid", "sigmoid", "tanh"])
    if kind == "small":
        # (one launch of the tanh variant holds up to 32 units at every row and feature count)
        return dict(kind=kind, n=rng.randint(40, 128), d=rng.randint(16, 48),
                    h=rng.randint(4, 32 if act == "tanh" else 64),
                    k=rng.randint(1, 4), epochs=_log(rng, 100, 1000), act=act, mu=rng.choice([0.0, 0.0, 0.9]))
    if kind == "autograd":
        return dict(kind=kind, n=_log(rng, 60, 50000), d=rng.randint(16, 64), h=_log(rng, 8, 256),
                    k=rng.randint(1, 4), act=act, dx=rng.random() < 0.3)
    if kind == "batched":
        return dict(kind=kind, nets=_log(rng, 64, 4000), d=rng.randint(24, 40), k=3, h_max=rng.choice([16, 32, 64]),
                    epochs=_log(rng, 20, 100))
    if kind == "readout":
        return dict(kind=kind, nets=_log(rng, 64, 4000), d=rng.randint(24, 40), k=3, h_max=rng.choice([16, 32, 64]))
    if kind == "minibatch":
        prec = rng.choice(["fp32", "fp32", "bf16", "e4m3"])
        batch = rng.choice([1024, 2048, 4096, 8192, 16384])
        h = rng.choice([128, 200, 256, 512, 777, 1024])
        steps = rng.randint(4, 64 if prec == "fp32" else 32)
        return dict(kind=kind, n=max(1, steps * batch - rng.randint(0, batch - 1)), d=rng.randint(24, 64), h=h, k=3,
                    batch=batch, prec=prec, epochs=1)
    if kind == "shared":
        return dict(kind=kind, nets=rng.choice([4, 8, 16, 32]), n=_log(rng, 30000, 130000), d=rng.choice([33, 48, 64]),
                    h=rng.choice([256, 512, 1024]), k=3, batch=rng.choice([4096, 8192, 16384]),
                    prec=rng.choice(["fp32", "bf16"]), epochs=1)
    if kind == "predict":
        return dict(kind=kind, n=_log(rng, 1000, 1000000), d=rng.randint(16, 64), h=_log(rng, 16, 256),
                    k=rng.randint(2, 4), act=act)
    if kind == "deep":
        return dict(kind=kind, n=rng.randint(40, 140), d=rng.randint(16, 40), h=rng.randint(8, 24),
                    h2=rng.randint(8, 24), k=3, act=act, epochs=_log(rng, 100, 500))
    return dict(kind=kind, n=_log(rng, 300, 20000), d=rng.randint(24, 64), h=_log(rng, 32, 256), h2=_log(rng, 16, 64),
                k=3, act=act, epochs=1)


# ------------------------------------------------------------------- inputs
def _rows(n, d, k, gen, device):
    """z-scored columns (two thirds Gaussian, the rest Bernoulli(0.3)) and
    the classes of a random teacher network, one-hot (k = 1: 0/1)."""
    x = torch.randn(n, d, generator=gen, device=device)
    nb = d // 3
    if nb:
        x[:, d - nb:] = (torch.rand(n, nb, generator=gen, device=device) < 0.3).float()
    x -= x.mean(0)
    x /= x.std(0, unbiased=False).clamp_min(0.05)
    w = torch.randn(8, d, generator=gen, device=device) / math.sqrt(d)
    score = torch.tanh(x @ w.t()) @ torch.randn(8, generator=gen, device=device)
    score = (score - score.mean()) / score.std(unbiased=False).clamp_min(1e-3)
    t = torch.zeros(n, k, device=device)
    if k == 1:
        t[:, 0] = (score >= 0.5).float()
    else:
        cls = torch.zeros(n, dtype=torch.long, device=device)
        for j in range(1, k):
            cls += (score >= -0.3 + 0.8 * (j - 1)).long()
        t.scatter_(1, cls[:, None], 1.0)
    return x.contiguous(), t


def _theta(count, gen, device):
    return torch.rand(count, generator=gen, device=device) - 0.5


def _gen(seed, device="cuda"):
    g = torch.Generator(device=device)
    g.manual_seed(1000003 * int(seed) + 17)
    return g


def _grid(case, held):
    """The network table: groups of five folds with a hidden size, a learning
    rate and 50..150 patients each; a net's own rows are four of the folds
    (`held`: the fifth).  It belongs to the case, the rows and the initial
    parameters to the seed."""
    g = torch.Generator()
    g.manual_seed(77 + case["nets"])
    items, row, p = [], 0, 0
    for i in range(case["nets"]):
        if i % 5 == 0:
            m = int(torch.randint(50, 151, (1,), generator=g))
            h = int(torch.randint(4, case["h_max"] + 1, (1,), generator=g))
            lr = float(10.0 ** (-2.0 + 2.0 * torch.rand(1, generator=g)))
        fold = m // 5 + (1 if i % 5 < m % 5 else 0)
        rows = fold if held else m - fold
        items.append(dict(n_rows=rows, n_hidden=h, lr=lr, x_off=row, p_off=p))
        row += rows
        p += case["d"] * h + h + h * case["k"] + case["k"]
    return items, row, p


def _lrs(nets):
    return [10.0 ** (-2.0 + 2.0 * (i % 8) / 7.0) for i in range(nets)]


def _inputs(case, seed):
    """The tensors of a case on the GPU, made from the seed alone."""
    dev, gen, kind = "cuda", _gen(seed), case["kind"]
    if kind in ("batched", "readout"):
        items, rows, p = _grid(case, kind == "readout")
        x, t = _rows(rows, case["d"], case["k"], gen, dev)
        return dict(X=x, T=t, items=items, theta=_theta(p, gen, dev))
    x, t = _rows(case["n"], case["d"], case["k"], gen, dev)
    d, h, k = case["d"], case["h"], case["k"]
    if kind in ("deep", "layers"):
        w = [d, h, case["h2"], k]
        return dict(X=x, T=t, theta=_theta(sum(w[i + 1] * (w[i] + 1) for i in range(3)), gen, dev))
    p = d * h + h + h * k + k
    if kind == "shared":
        return dict(X=x, T=t, theta=_theta(case["nets"] * p, gen, dev).view(case["nets"], p))
    return dict(X=x, T=t, theta=_theta(p, gen, dev))


def prepare(case, seed):
    s = _inputs(case, seed)
    kind, dev = case["kind"], "cuda"
    s["case"] = case
    if kind in ("batched", "readout"):
        s["plan"] = mlp.BatchPlan(s["items"], buckets=kind == "batched")
        if kind == "batched":
            s["comp"] = torch.zeros_like(s["theta"])
            s["hist"] = torch.empty(case["nets"], case["epochs"], device=dev)
        else:
            s["group"] = torch.arange(case["nets"], device=dev, dtype=torch.int32) // 5
        return s
    d, h, k = case["d"], case["h"], case["k"]
    host = s["theta"].cpu().numpy()
    if kind in ("deep", "layers"):
        s["net"] = mlp.DeepNet([d, h, case["h2"], k], theta=host, act=case["act"], lr=LR)
        s["hist"] = torch.empty(case["epochs"], device=dev)
    elif kind == "shared":
        s["comp"] = torch.zeros_like(s["theta"])
        s["hist"] = torch.empty(case["nets"], case["epochs"], device=dev)
        s["ws"] = torch.empty(mlp.shared_workspace_size(d, h, k, case["n"], case["batch"], case["nets"], case["prec"]),
                              dtype=torch.uint8, device=dev)
    else:
        # a network that predicts a table was trained on it in minibatches
        batch = min(case["n"], 4096) if kind == "predict" else case.get("batch", 0)
        s["net"] = mlp.Net(d, h, k, case["n"], batch=batch, lr=LR, prec=case.get("prec", "fp32"),
                           theta=host, act=case.get("act", "sigmoid"), momentum=case.get("mu", 0.0))
        if kind in ("small", "minibatch"):
            s["hist"] = torch.empty(case["epochs"], device=dev)
        if kind == "autograd":
            net = s["net"]
            s["params"] = [v.requires_grad_(True) for v in (net.W1, net.b1, net.W2, net.b2)]
            s["X"].requires_grad_(case["dx"])
    return s


def run(s):
    """Trained parameters and losses (the compensation terms, which hold the
    rounding errors of the update, are no result); gradients; outputs."""
    case = s["case"]
    kind, X, T = case["kind"], s["X"], s["T"]
    if kind in ("small", "minibatch"):
        s["net"].train(X, T, case["epochs"], loss_hist=s["hist"])
        return dict(theta=s["net"].flat, loss=s["hist"])
    if kind == "autograd":
        net, params = s["net"], s["params"]
        Y = mlp.MLPFunction.apply(net, X, *params)
        loss = torch.nn.functional.mse_loss(Y, T)
        grads = torch.autograd.grad(loss, params + ([X] if case["dx"] else []))
        with torch.no_grad():
            net.step(mlp.Grads(*grads[:4], None))
        return dict(Y=Y, loss=loss, grads=list(grads), theta=net.flat)
    if kind == "batched":
        mlp.train_batched(s["plan"], X, T, s["theta"], s["comp"], case["epochs"], case["d"], case["k"],
                          loss_hist=s["hist"])
        return dict(theta=s["theta"], loss=s["hist"])
    if kind == "readout":
        loss, correct = mlp.eval_batched(s["plan"], X, T, s["theta"], case["d"], case["k"])
        mean, best = mlp.cv_select(loss, s["group"], (case["nets"] + 4) // 5)
        return dict(loss=loss, correct=correct, mean=mean, best=best)
    if kind == "shared":
        mlp.train_shared(X, T, s["theta"], _lrs(case["nets"]), case["epochs"], case["h"], batch=case["batch"],
                         prec=case["prec"], comp=s["comp"], loss_hist=s["hist"], workspace=s["ws"])
        return dict(theta=s["theta"], loss=s["hist"])
    if kind == "predict":
        Y, labels, correct = s["net"].predict(X, T)
        return dict(Y=Y, labels=labels, correct=correct)
    train = s["net"].train_kernel if kind == "deep" else s["net"].train_fused
    train(X, T, case["epochs"], loss_hist=s["hist"])
    return dict(theta=s["net"].flat, loss=s["hist"])


# --------------------------------------------------------------------- work
def _net_flops(d, h, k):
    """Training flops of one row: forward, error, deltas, gradients."""
    return 4 * d * h + 6 * h * k + 7 * h + 11 * k


def work(case):
    """One pass: every input read once (also where several epochs read it),
    every output written once; the method's floating-point operations."""
    kind, d, k = case["kind"], case["d"], case["k"]
    if kind in ("batched", "readout"):
        items, rows, p = _grid(case, kind == "readout")
        if kind == "readout":
            fl = sum(it["n_rows"] * (2 * d * it["n_hidden"] + (2 * k + 4) * it["n_hidden"] + 7 * k) for it in items)
            return dict(bytes=4 * (rows * (d + k) + p + 3 * case["nets"]), flops=fl)
        e = case["epochs"]
        fl = sum(it["n_rows"] * _net_flops(d, it["n_hidden"], k) for it in items) + 2 * p
        return dict(bytes=4 * (rows * (d + k) + 2 * p + case["nets"] * e), flops=fl * e)
    n, h = case["n"], case["h"]
    p = d * h + h + h * k + k
    if kind in ("deep", "layers"):
        w = [d, h, case["h2"], k]
        p = sum(w[i + 1] * (w[i] + 1) for i in range(3))
        per = sum(4 * w[i] * w[i + 1] + 4 * w[i + 1] for i in range(3)) + sum(2 * w[i] * w[i + 1] for i in (1, 2))
        return dict(bytes=4 * (n * (d + k) + 2 * p), flops=case["epochs"] * (n * per + 2 * p))
    if kind == "predict":
        return dict(bytes=4 * (n * (d + k) + p + n * (k + 1)), flops=n * (2 * d * h + (2 * k + 4) * h + 4 * k))
    if kind == "autograd":
        dx = 2 * d * h if case["dx"] else 0
        return dict(bytes=4 * (n * (d + 2 * k) + 3 * p + (n * d if case["dx"] else 0)),
                    flops=n * (_net_flops(d, h, k) + dx) + 2 * p)
    m = case.get("nets", 1)
    steps = math.ceil(n / case["batch"]) if case.get("batch") else 1
    return dict(bytes=4 * (n * (d + k) + 2 * m * p), flops=m * case["epochs"] * (n * _net_flops(d, h, k) + 2 * p * steps))


# -------------------------------------------------------------------- exact
def _split(flat, d, h, k):
    a, b, c = d * h, d * h + h, d * h + h + k * h
    return flat[:a].view(h, d), flat[a:b], flat[b:c].view(k, h), flat[c:]


def _act(z, act):
    return torch.tanh(z) if act == "tanh" else torch.sigmoid(z)


def _slope(a, act):
    return 1 - a * a if act == "tanh" else a * (1 - a)


def _grad(X, T, flat, shape, act, want_dx=False):
    """(loss, packed gradient, Y, dX) of one network in float64."""
    W1, b1, W2, b2 = _split(flat, *shape)
    A = _act(X @ W1.t() + b1, act)
    Y = torch.sigmoid(A @ W2.t() + b2)
    err = Y - T
    d2 = 2 * err / err.numel() * Y * (1 - Y)
    d1 = (d2 @ W2) * _slope(A, act)
    g = torch.cat([(d1.t() @ X).reshape(-1), d1.sum(0), (d2.t() @ A).reshape(-1), d2.sum(0)])
    return (err * err).mean(), g, Y, (d1 @ W1 if want_dx else None)


def _descend(X, T, flat, shape, lr, epochs, batch, act="sigmoid", mu=0.0):
    n = X.shape[0]
    b = batch if 0 < batch < n else n
    vel, losses = torch.zeros_like(flat), []
    for _ in range(epochs):
        per = []
        for r in range(0, n, b):
            loss, g, _, _ = _grad(X[r:r + b].double(), T[r:r + b].double(), flat, shape, act)
            vel = mu * vel + g
            flat = flat - lr * vel
            per.append(loss)
        losses.append(torch.stack(per).mean())
    return flat, torch.stack(losses)


def _pad(s, case):
    """The packed networks as one padded batch: rows, masks, parameters."""
    items, d, k = s["items"], case["d"], case["k"]
    m, N, H = len(items), max(it["n_rows"] for it in items), max(it["n_hidden"] for it in items)
    dev = s["X"].device
    nr = torch.tensor([it["n_rows"] for it in items], device=dev)
    nh = torch.tensor([it["n_hidden"] for it in items], device=dev)
    xo = torch.tensor([it["x_off"] for it in items], device=dev)
    po = torch.tensor([it["p_off"] for it in items], device=dev)
    r, u = torch.arange(N, device=dev), torch.arange(H, device=dev)
    rm, hm = r[None] < nr[:, None], u[None] < nh[:, None]
    idx = torch.where(rm, xo[:, None] + r[None], xo[:, None])
    X = s["X"].double()[idx] * rm[..., None]
    T = s["T"].double()[idx] * rm[..., None]
    i1 = po[:, None, None] + u[None, :, None] * d + torch.arange(d, device=dev)[None, None]
    ib1 = (po + nh * d)[:, None] + u[None]
    i2 = (po + nh * (d + 1))[:, None, None] + torch.arange(k, device=dev)[None, :, None] * nh[:, None, None] + u
    ib2 = (po + nh * (d + 1 + k))[:, None] + torch.arange(k, device=dev)[None]
    masks = [hm[..., None].expand_as(i1), hm, hm[:, None].expand_as(i2), torch.ones_like(ib2, dtype=torch.bool)]
    th = s["theta"].double()
    idx4 = [i1, ib1, i2, ib2]
    pars = [torch.where(q, th[torch.where(q, i, 0)], 0.0) for i, q in zip(idx4, masks)]
    lr = torch.tensor([it["lr"] for it in items], device=dev, dtype=torch.float32).double()
    return X, T, rm, hm, nr, pars, idx4, masks, lr


def _forward_many(X, pars, hm):
    W1, b1, W2, b2 = pars
    A = torch.sigmoid(torch.bmm(X, W1.transpose(1, 2).contiguous()) + b1[:, None]) * hm[:, None]
    return A, torch.sigmoid(torch.bmm(A, W2.transpose(1, 2).contiguous()) + b2[:, None])


def _classes(v):
    return (v[..., 0] > 0.5).int() if v.shape[-1] == 1 else v.argmax(-1).int()


def exact(case, seed):
    s = _inputs(case, seed)
    kind, d, k = case["kind"], case["d"], case["k"]
    if kind in ("batched", "readout"):
        X, T, rm, hm, nr, pars, idx4, masks, lr = _pad(s, case)
        scale = 1.0 / (nr.double() * k)
        if kind == "readout":
            _, Y = _forward_many(X, pars, hm)
            loss = (((Y - T) ** 2) * rm[..., None]).sum((1, 2)) * scale
            mean = torch.stack([v.mean() for v in loss.split(5)])
            return dict(loss=loss, correct=None, mean=mean, best=None)
        Xt = X.transpose(1, 2).contiguous()
        for _ in range(case["epochs"]):
            A, Y = _forward_many(X, pars, hm)
            err = (Y - T) * rm[..., None]
            d2 = 2 * err * scale[:, None, None] * Y * (1 - Y)
            d1 = torch.bmm(d2, pars[2]) * A * (1 - A)
            grads = [torch.bmm(Xt, d1).transpose(1, 2), d1.sum(1),
                     torch.bmm(d2.transpose(1, 2).contiguous(), A), d2.sum(1)]
            pars = [q - lr.view(-1, *([1] * (q.dim() - 1))) * g for q, g in zip(pars, grads)]
        th = s["theta"].double()
        for q, i, msk in zip(pars, idx4, masks):
            th[i[msk]] = q[msk]
        # the loss rows come in the launch order the plan chose: no fixed value
        return dict(theta=th, loss=None)
    X, T, th, h = s["X"], s["T"], s["theta"].double(), case["h"]
    if kind in ("small", "minibatch"):
        flat, loss = _descend(X, T, th, (d, h, k), LR, case["epochs"], case.get("batch", 0),
                              case.get("act", "sigmoid"), case.get("mu", 0.0))
        return dict(theta=flat, loss=loss)
    if kind == "shared":
        got = [_descend(X, T, th[i], (d, h, k), lr, case["epochs"], case["batch"])
               for i, lr in enumerate(torch.tensor(_lrs(case["nets"])).double().tolist())]
        return dict(theta=torch.stack([g[0] for g in got]), loss=torch.stack([g[1] for g in got]))
    if kind == "autograd":
        loss, g, Y, dX = _grad(X.double(), T.double(), th, (d, h, k), case["act"], case["dx"])
        return dict(Y=Y, loss=loss, grads=list(_split(g, d, h, k)) + ([dX] if case["dx"] else []), theta=th - LR * g)
    if kind == "predict":
        W1, b1, W2, b2 = _split(th, d, h, k)
        return dict(Y=torch.sigmoid(_act(X.double() @ W1.t() + b1, case["act"]) @ W2.t() + b2), labels=None,
                    correct=None)
    # several hidden layers: torch's own derivatives
    w, off, layers = [d, h, case["h2"], k], 0, []
    for i in range(3):
        c = w[i + 1] * w[i]
        layers += [th[off:off + c].view(w[i + 1], w[i]).clone(), th[off + c:off + c + w[i + 1]].clone()]
        off += c + w[i + 1]
    X, T, losses = X.double(), T.double(), []
    for _ in range(case["epochs"]):
        layers = [v.detach().requires_grad_(True) for v in layers]
        a = X
        for i in range(3):
            a = _act(a @ layers[2 * i].t() + layers[2 * i + 1], case["act"] if i < 2 else "sigmoid")
        loss = torch.nn.functional.mse_loss(a, T)
        grads = torch.autograd.grad(loss, layers)
        layers = [v.detach() - LR * g for v, g in zip(layers, grads)]
        losses.append(loss.detach())
    return dict(theta=torch.cat([v.reshape(-1) for v in layers]), loss=torch.stack(losses))
