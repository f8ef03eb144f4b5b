"""mlp_backward on both sides of the rules that choose
the form of the gradient sums, against float64 with the bounds of
test_gpu_grads."""
import pytest

from test_gpu_grads import M, test_backward_edges as backward   # noqa: F401

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
])
def test_backward_forms(M, n, d, h, k, act, mse):   # noqa: F811
    backward(M, n, d, h, k, act, mse)
