"""Maps whose columns do not fill the last group of eight (every remainder; fewer than eight columns; a last group that begins a
strip), over the shapes of the reduction's workgroups and head counts that leave every size of a last batch."""
import pytest
import torch

from paper_2411_17686_amd import ficoco as fc
from paper_2411_17686_amd import synth
from tests import parity as P

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = fc.Context(0)
    yield c
    c.close()


def case(N, B, H, dtype):
    cfg = synth.ficoco_v_single(seed=N + B + H, B=B, grid=1, D=16, H=H, centres=7, dtype=dtype, n_keep=max(1, N // 2))
    g = torch.Generator().manual_seed(N * H + B)
    cfg["X"] = torch.randn(B, N + 1, 16, generator=g).to(cfg["X"].dtype)
    cfg["A"] = torch.softmax(torch.randn(B, H, N + 1, N + 1, generator=g), -1).to(cfg["A"].dtype)
    cfg["N"], cfg["grid"] = N, (1, 1, N)
    return cfg


# tokens, images, heads; workgroups of 8 x 24 lanes and groups (up to 256 tokens, few of them), 16 x 16 and 32 x 8
CASES = [(n, 2, 3) for n in (3, 7, 8, 9, 15, 18, 65, 193)] + [(n, 3, 5) for n in (129, 190, 194, 197, 199, 202)] \
    + [(150, 40, 2), (129, 48, 5), (257, 70, 1), (253, 70, 3)] + [(n, 1, h) for n, h in ((257, 1), (259, 9), (262, 13), (321, 17), (519, 16), (577, 20))] \
    + [(261, 64, 4), (386, 48, 3), (1029, 3, 2)]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("N,B,H", CASES)
def test_ragged_columns(ctx, N, B, H, dtype):
    cfg = case(N, B, H, dtype)
    for corr in (fc.C_ATTN, fc.C_COSINE) if B < 8 else (fc.C_ATTN,):
        kw = dict(red_src=fc.R_ATTN_RECV, sem_src=fc.G_CLS_ATTN, corr_src=corr)
        out, _ = P.run_v(cfg, cfg["A"], ctx=ctx, **kw)
        for b in {0, B // 2, B - 1}:
            P.compare_image(out, b, P.oracle_v(cfg, cfg["A"], b, **kw), dtype, cfg["vis_begin"], corr == fc.C_ATTN)


# Heads of one row a thread: whole batches of eight and sixteen, one head past them, what is left of each size; text rows alike.
HEADS = [16, 17, 20, 23, 24, 25, 29, 33, 40]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("H", HEADS)
def test_heads_of_one_row(ctx, H, dtype):
    cfg = case(72, 2, H, dtype)
    for corr in (fc.C_ATTN, fc.C_COSINE):
        kw = dict(red_src=fc.R_ATTN_RECV, sem_src=fc.G_CLS_ATTN, corr_src=corr)
        out, _ = P.run_v(cfg, cfg["A"], ctx=ctx, **kw)
        for b in range(2):
            P.compare_image(out, b, P.oracle_v(cfg, cfg["A"], b, **kw), dtype, cfg["vis_begin"], corr == fc.C_ATTN)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("H", HEADS)
def test_heads_of_text_rows(ctx, H, dtype):
    cfg = synth.ficoco_l_decoder(seed=H, B=2, n_sys=3, N=72, M=9, D=32, H=H, centres=7, n_keep=24, dtype=dtype, with_vv=True)
    for red, corr in ((fc.R_ATTN_RECV, fc.C_ATTN), (fc.R_SIM_MEAN, fc.C_COSINE)):
        out, _ = P.run_l(cfg, red, corr, ctx=ctx)
        for b in range(2):
            P.compare_image(out, b, P.oracle_l(cfg, b, red, corr), dtype, cfg["vis_begin"], False)
