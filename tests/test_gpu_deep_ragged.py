"""One-launch training of several hidden layers where one of 33..64 units is
among narrower ones, whose padding tiles are skipped, against the FP64 oracle."""
import pytest

from test_gpu_deep_tiles import M, test_tiled_deep_training_matches_the_oracle as against_oracle   # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("widths,rows,act,epochs", [
    ([4, 8, 4, 48, 1], 3, "sigmoid", 200),       # widest layer last
    ([10, 49, 3, 2], 37, "tanh", 100),           # ... first, one unit past a tile
    ([33, 16, 64, 17, 3], 16, "sigmoid", 100),   # ... between, one and two tiles beside it
    ([20, 33, 17, 5], 30, "tanh", 100),          # three tiles, two, one
    ([5, 40, 4], 60, "sigmoid", 100),            # one hidden layer of three tiles of four
    ([16, 33, 50, 50, 2], 16, "sigmoid", 100),   # too little padding: nothing skipped
    ([4, 40, 4, 4], 80, "sigmoid", 100),
])
def test_ragged_layers(M, widths, rows, act, epochs):   # noqa: F811
    against_oracle(M, widths, rows, act, epochs)
