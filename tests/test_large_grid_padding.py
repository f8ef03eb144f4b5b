"""The default grid in float32 does not take a split whose hidden blocks are
padded to more rows x units than another of as many workgroups."""
import pytest

from paper_1908_07847_amd import mlp


def grids(h, b, prec):
    """Every grid of the default rule's kind: (workgroups, padded work, grid)."""
    out, gj = [], 1
    while -(-h // (64 * gj)) * 64 > 256:
        gj *= 2
    first = gj
    while gj <= 16 and (gj == first or h > 64 * (gj // 2)):
        gi = 1
        while gi * gj <= 256 and b % (gi * 32) == 0 and (b // gi >= 64 or gi <= (128 if prec == "fp32" else 32)):
            out.append((gi * gj, b // gi * (-(-h // (64 * gj)) * 64), (gi, gj)))
            gi *= 2
        gj *= 2
    return out


@pytest.mark.parametrize("h,b,want", [(129, 16384, (256, 1)), (192, 16384, (256, 1)), (384, 8192, (128, 2)),
                                      (768, 4096, (64, 4)), (1500, 2048, (32, 8)),
                                      (256, 4096, (64, 4)), (512, 8192, (64, 4)), (777, 4096, (32, 8))])
def test_fp32_grid_counts_the_padding(h, b, want):
    p = mlp.large_plan(33, h, 3, 4 * b, batch=b, prec="fp32", n_cu=256)
    assert (p["row_blocks"], p["hidden_blocks"]) == want


def test_fp32_grid_is_never_more_work():
    for h in list(range(1, 1100, 37)) + [64, 129, 192, 257, 384, 513, 768, 1500, 3000, 4096]:
        for b in (32, 96, 256, 1024, 2048, 4096, 8192, 16384, 32768):
            p = mlp.large_plan(33, h, 3, 4 * b, batch=b, prec="fp32", n_cu=256)
            all_ = grids(h, b, "fp32")
            most = max(g[0] for g in all_)
            assert p["row_blocks"] * p["hidden_blocks"] == most
            units = -(-h // (64 * p["hidden_blocks"])) * 64
            assert b // p["row_blocks"] * units == min(g[1] for g in all_ if g[0] == most), (h, b, p)


@pytest.mark.parametrize("prec", ["bf16", "e4m3"])
def test_reduced_precisions_stay_square(prec):
    p = mlp.large_plan(33, 192, 3, 65536, batch=16384, prec=prec, n_cu=256)
    assert (p["row_blocks"], p["hidden_blocks"]) == (128, 2)
