"""mlp_backward and mlp_dense_backward on both sides of the rules that choose
the form of the gradient sums, against float64 with the bounds of
test_gpu_grads."""
import pytest

from test_gpu_grads import M, test_backward_edges as backward, test_dense_backward_edges as dense   # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,h,k,act,mse", [
    (1, 1, 1, 4, "tanh", True),
    (64, 64, 16, 1, "sigmoid", True),      # one wave's rows exactly
    (65, 65, 17, 3, "sigmoid", False),     # one row and one input past it
    (513, 130, 20, 4, "tanh", True),       # a second set for one wave, three input tiles
    (2048, 48, 195, 4, "sigmoid", True),   # the most rows and work of the few-rows form ...
    (2048, 48, 196, 4, "sigmoid", True),
    (2049, 10, 10, 1, "sigmoid", False),   # ... and one past each
    (780, 64, 512, 2, "sigmoid", False),
    (700, 64, 513, 2, "tanh", True),       # more units than resident workgroups
    (1024, 20, 30, 5, "sigmoid", True),    # more than four outputs: fewer rows
    (1025, 20, 30, 5, "sigmoid", False),
    (300, 33, 700, 3, "sigmoid", True),    # tiles in three ranges
    (129, 200, 300, 16, "tanh", False),    # ... in two, the second of one row
])
def test_backward_forms(M, n, d, h, k, act, mse):   # noqa: F811
    backward(M, n, d, h, k, act, mse)


@pytest.mark.parametrize("n,din,dout,act", [
    (128, 100, 700, 1), (129, 100, 700, 0),    # one range and two, two input tiles
    (3000, 130, 70, 0),                        # three ragged input tiles, partials of every range
    (4100, 700, 40, 1),                        # the workspace limits the ranges to five
    (2100, 2200, 20, 0),                       # ... to one
    (2049, 64, 64, 1), (2300, 33, 16, 0),      # ranges of 128 rows
])
def test_dense_forms(M, n, din, dout, act):   # noqa: F811
    dense(M, n, din, dout, act)
