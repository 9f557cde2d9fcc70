"""Where norms, unit rows and column sums of a decoder's features are one pass over the tokens (host code; nothing is launched)."""
import pytest

from paper_2411_17686_amd import ficoco as fc
from tests import plan_hook as H

# sequences, visual tokens, text tokens, features, us of the step in one pass and in separate ones
MEASURED = [(8, 690, 64, 5120, (145.8, 151.8)), (12, 690, 64, 5120, (184.5, 183.9)), (8, 1152, 64, 5120, (221.2, 214.6)), (8, 1152, 200, 5120, (252.3, 241.1)),
            (16, 576, 200, 5120, (237.1, 231.7)), (8, 1152, 64, 4096, (170.8, 179.7)), (8, 1152, 200, 6144, (284.0, 283.3)),
            (32, 200, 200, 8192, (253.3, 263.6)), (24, 576, 200, 8192, (455.7, 486.7)), (64, 64, 200, 8192, (263.6, 251.2)), (128, 33, 200, 8192, (414.4, 393.4))]


# the same with the correlation by attention: no unit rows are wanted
BY_ATTENTION = [(7, 585, 2, 8192, (142.8, 130.3)), (21, 210, 5, 7168, (139.8, 128.7)), (12, 364, 24, 6144, (124.7, 119.0)), (8, 526, 12, 5120, (123.7, 116.6)),
                (16, 195, 32, 6144, (86.6, 93.7)), (6, 426, 10, 8192, (99.9, 101.2)), (5, 1023, 4, 4096, (121.7, 122.9)), (15, 434, 4, 8192, (168.5, 159.4))]


@pytest.mark.parametrize("B,N,M,D,us,corr", [m + (fc.C_COSINE,) for m in MEASURED] + [m + (fc.C_ATTN,) for m in BY_ATTENTION])
def test_one_pass_where_it_is_faster(B, N, M, D, us, corr):
    p = fc.Problem()
    p.variant, p.dtype, p.red_src, p.sem_src, p.corr_src = fc.VARIANT_L, fc.BF16, fc.R_SIM_MEAN, fc.G_TEXT_ATTN, corr
    p.B, p.N, p.M, p.D, p.A_text = B, N, M, D, 4096
    assert us[0 if H.unit_rows_summed(p) else 1] <= 1.01 * min(us)
