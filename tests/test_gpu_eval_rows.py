"""Evaluation of networks of up to 16 units, whose waves split the rows, and of
the shapes that go to one thread per row, against float64."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,k,shapes,copies", [
    (1, 1, [(1, 1), (31, 2), (300, 6)], 1),              # a thread per row
    (1, 3, [(1, 1), (33, 16), (300, 16)], 1),            # ... and past its work
    (4, 4, [(32, 16), (33, 15), (129, 1), (1000, 10)], 1),   # one set, two, a second round, many
    (33, 3, [(25, 4), (60, 16), (64, 9), (128, 16), (97, 3)], 1),
    (64, 2, [(40, 16), (4200, 12)], 1),                  # the longest contraction; sums in two levels
    (33, 3, [(25, 17), (60, 9)], 1),                     # one network too wide: tiles over the waves
    (2, 3, [(96, 12), (3, 1)], 700),                     # many networks: a thread per row
    (3, 3, [(96, 11), (3, 1)], 700),
    (1, 2, [(256, 40), (5, 2)], 700),
])
def test_eval_forms(d, k, shapes, copies):
    from paper_1908_07847_amd import mlp
    print(f"eval d={d} k={k} {shapes} x {copies}", flush=True)
    g = np.random.default_rng(d + len(shapes))
    items, xs, ts, th, row, off, ref = [], [], [], [], 0, 0, []
    for n, h in shapes * copies:
        X = g.normal(size=(n, d)).astype(np.float32)
        T = np.zeros((n, k), np.float32)
        T[np.arange(n), g.integers(0, k, n)] = g.integers(0, 2, n) if k == 1 else 1.0
        p = g.uniform(-0.5, 0.5, d * h + h + h * k + k).astype(np.float32)
        items.append(dict(n_rows=n, n_hidden=h, lr=0.0, x_off=row, p_off=off))
        W1, b1 = p[:d * h].reshape(h, d).astype(np.float64), p[d * h:d * h + h].astype(np.float64)
        A = 1 / (1 + np.exp(-(X.astype(np.float64) @ W1.T + b1)))
        Y = 1 / (1 + np.exp(-(A @ p[d * h + h:-k].reshape(k, h).T.astype(np.float64) + p[-k:])))
        cls = lambda v: (v[:, 0] > 0.5) if k == 1 else v.argmax(1)
        srt = np.sort(Y, 1)
        near = int(((np.abs(Y[:, 0] - 0.5) if k == 1 else srt[:, -1] - srt[:, -2]) < 1e-5).sum())
        ref.append((np.mean((Y - T) ** 2), int((cls(Y) == cls(T)).sum()), near))
        xs.append(X), ts.append(T), th.append(p)
        row, off = row + n, off + p.size
    plan = mlp.BatchPlan(items)
    cat = lambda v: torch.from_numpy(np.concatenate(v)).cuda()
    loss, correct = (v.cpu().numpy() for v in mlp.eval_batched(plan, cat(xs), cat(ts), cat(th), d, k))
    for i, (l, c, near) in enumerate(ref):
        # an output is within (d + h + 8) u of its sums' size, below 1e-5 here
        assert abs(float(loss[i]) - l) <= 2e-5 * l + 1e-9, (i, float(loss[i]), l)
        assert abs(int(correct[i]) - c) <= near, (i, int(correct[i]), c)
