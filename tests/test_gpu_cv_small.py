"""Selection over few nets, one launch up to 128 nets and 4096 groups, on both
sides of that rule, and where means tie or are not finite."""
import numpy as np
import pytest
import torch

from test_gpu_forward import M, test_cv_select_group_waves as select   # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,ng", [(1, 1), (5, 17), (64, 1), (65, 15), (100, 16), (128, 1000), (128, 1025), (128, 4096),
                                  (128, 4097), (129, 4096)])
def test_few_nets(M, n, ng):   # noqa: F811
    select(M, n, ng)


@pytest.mark.parametrize("ng", [3, 40, 2000, 5000])
def test_ties_and_non_finite(M, ng):   # noqa: F811
    loss = np.array([np.nan, 0.25, np.inf, 0.25, 0.5], np.float32)
    group = np.array([0, 2, 1, ng - 1, 1], np.int32)
    mean, best = M.cv_select(torch.from_numpy(loss).cuda(), torch.from_numpy(group).cuda(), ng)
    torch.cuda.synchronize()
    want = np.full(ng, np.inf, np.float32)
    want[2] = want[ng - 1] = 0.25
    assert np.array_equal(mean.cpu().numpy(), want)
    assert int(best) == 2      # the lowest index of the ties
    mean, best = M.cv_select(torch.full((2,), float("nan"), device="cuda"),
                             torch.tensor([1, 2], dtype=torch.int32, device="cuda"), ng)
    assert int(best) == 0 and bool(torch.isinf(mean).all())
