"""A batched net's result and its company: the same bits in any company and
order under a launch hint that fixes the shape, and without one as long as
the shape stays; across the shapes the library picks by itself, the FP64
oracle's result either way."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    from paper_1908_07847_amd import mlp
    return mlp


D, K, EPOCHS = 33, 3, 40


def nets_of(widths, rows):
    """Nets with data and parameters that depend on their index alone."""
    out = []
    for i, (h, n) in enumerate(zip(widths, rows)):
        g = np.random.default_rng(1000 + i)
        X = g.normal(size=(n, D)).astype(np.float32)
        T = np.zeros((n, K), np.float32)
        T[np.arange(n), g.integers(0, K, n)] = 1.0
        out.append((h, X, T, g.uniform(-0.5, 0.5, D * h + h + h * K + K).astype(np.float32)))
    return out


def train(M, nets, hint=0):
    items, off, row = [], 0, 0
    for h, X, _, th in nets:
        items.append(dict(n_rows=len(X), n_hidden=h, lr=0.1, x_off=row, p_off=off))
        row, off = row + len(X), off + th.size
    cat = lambda j: torch.from_numpy(np.concatenate([n[j] for n in nets])).cuda()
    theta = cat(3)
    try:
        M.set_launch_hint(small_threads=hint)
        M.train_batched(M.BatchPlan(items), cat(1), cat(2), theta, torch.zeros_like(theta), EPOCHS, D, K)
        torch.cuda.synchronize()
    finally:
        M.reset_launch_hint()
    t = theta.cpu().numpy()
    return [t[it["p_off"]:it["p_off"] + n[3].size] for it, n in zip(items, nets)]


FEW = nets_of([10, 16, 5, 30, 9], [60, 120, 33, 97, 128])
SMALL = nets_of([10, 16, 5, 30, 9] + [8] * 300, [60, 120, 33, 97, 128] + [20] * 300)   # above one net per CU
WIDE = SMALL + nets_of([64], [128])                                                    # ... and one wider than 32 units


@pytest.mark.parametrize("hint", [64, 128])
def test_fixed_shape_gives_the_same_bits_in_any_company(M, hint):
    print(f"company under hint {hint}", flush=True)
    few, small, wide = (train(M, n, hint) for n in (FEW, SMALL, WIDE))
    turned = train(M, WIDE[::-1], hint)[::-1]
    for i in range(len(FEW)):
        for other in (small, wide, turned):
            assert np.array_equal(few[i], other[i]), i


def test_default_shapes(M):
    print("company without a hint", flush=True)
    few, small, wide = (train(M, n) for n in (FEW, SMALL, WIDE))
    more = train(M, SMALL + nets_of([32, 1], [128, 1]))      # the shape stays
    for i in range(len(SMALL)):
        assert np.array_equal(small[i], more[i]), i
    for i, (h, X, T, th) in enumerate(FEW):
        q, _ = oracle.train(X, T, oracle.Params.of(unpack(th, h)), 0.1, EPOCHS)
        ref = np.concatenate([q.W1.ravel(), q.b1, q.W2.ravel(), q.b2])
        for got in (few[i], small[i], wide[i]):
            assert np.max(np.abs(got - ref)) <= 1e-5 * np.max(np.abs(ref))     # the trainers' stated tolerance


def unpack(th, h):
    from paper_1908_07847_amd import synth
    return synth.Theta.unpack(th, D, h, K)
