"""The large-N trainer's default grid: what every choice has to satisfy, and
that a shape is refused only where no grid of one workgroup per CU covers it."""
import pytest

from paper_1908_07847_amd import mlp


@pytest.mark.parametrize("prec", ["fp32", "bf16", "e4m3"])
@pytest.mark.parametrize("n_cu", [1, 5, 64, 256, 304])
def test_default_grid(prec, n_cu):
    for h in (1, 64, 65, 200, 256, 257, 777, 1024, 3000, 4096):
        for b in (32, 96, 256, 1024, 1536, 2048, 4096, 8192, 16384, 32 * 33, 32 * 8191):
            need = 1
            while -(-h // (64 * need)) * 64 > 256:
                need *= 2
            if need > n_cu:
                with pytest.raises(Exception):
                    mlp.large_plan(33, h, 3, b, batch=b, prec=prec, n_cu=n_cu)
                continue
            p = mlp.large_plan(33, h, 3, b, batch=b, prec=prec, n_cu=n_cu)
            gi, gj = p["row_blocks"], p["hidden_blocks"]
            rows, units = b // gi, -(-h // (64 * gj)) * 64
            assert gi * gj <= min(n_cu, 256) and gi <= 256 and gj <= 16
            assert rows * gi == b and rows % 32 == 0 and 64 <= units <= 256
            assert rows % p["piece_rows"] == 0
            if rows < 64:
                assert gi <= (128 if prec == "fp32" else 32)
            # twice the row blocks would not have fitted with this split
            assert (2 * gi * gj > min(n_cu, 256) or rows % 64 or
                    (rows // 2 < 64 and 2 * gi > (128 if prec == "fp32" else 32)))
