"""A decoder call with visual maps reads the text block in the launch of the maps: widths below, at and above the
columns of a strip and of a text workgroup, text rows below, at and above its eight."""
import pytest

from paper_2411_17686_amd import ficoco as fc
from paper_2411_17686_amd import synth
from tests import parity as P

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = fc.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("N", [7, 64, 65, 130, 191, 192, 193, 256, 257, 400, 600])
@pytest.mark.parametrize("M,dtype", [(1, "f32"), (8, "bf16"), (9, "bf16"), (35, "f32")])
def test_maps_and_text(ctx, N, M, dtype):
    cfg = synth.ficoco_l_decoder(seed=N + M, B=2, n_sys=3, N=N, M=M, D=32, H=3, centres=5, n_keep=max(1, N // 3),
                                 dtype=dtype, with_vv=True)
    for red, corr, staged in ((fc.R_ATTN_RECV, fc.C_ATTN, False), (fc.R_ATTN_RECV, fc.C_COSINE, True)):
        out, _ = P.run_l(cfg, red, corr, k_max=64, ctx=ctx, staged=staged)
        for b in range(2):
            P.compare_image(out, b, P.oracle_l(cfg, b, red, corr), dtype, cfg["vis_begin"], False)
