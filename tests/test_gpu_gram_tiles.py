"""Cosine correlation of batches with many tiles of approximate values (128 x 128, 192 x 192 or 256 x 192, by an estimate of their
time): rows and columns that fill a tile, miss it by one and pass it by one, feature counts of less than a stage, whole
stages and stages with a remainder, several K ranges.  These are outputs of whole steps; the tiles' own values, which
outputs need not show, are compared in test_gpu_gram_block.py."""
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


# images, side of the grid, kept tokens (the others are the rows of the product), features
CASES = [(128, 15, 33, 8), (128, 15, 34, 72), (64, 15, 32, 136), (33, 20, 193, 200), (64, 20, 190, 256), (128, 15, 33, 320),
         (129, 17, 33, 64), (129, 17, 34, 192), (130, 17, 35, 328), (150, 16, 40, 24), (65, 21, 193, 128),
         # several K ranges: 288 and 232 features, 416 and 360, eight of which the last has 40
         (64, 19, 169, 520), (64, 19, 170, 776), (16, 19, 169, 2056), (24, 24, 192, 1032)]


@pytest.mark.parametrize("B,grid,n_keep,D", CASES)
def test_wide_tiles(ctx, B, grid, n_keep, D):
    cfg = synth.ficoco_v_single(seed=900 + D + n_keep, B=B, grid=grid, D=D, H=1, centres=7, dtype="bf16", n_keep=n_keep)
    kw = dict(red_src=fc.R_ATTN_RECV, sem_src=fc.G_CLS_ATTN, corr_src=fc.C_COSINE)
    out, _ = P.run_v(cfg, cfg["A"], ctx=ctx, k_max=16, **kw)
    for b in (0, B // 2, B - 1):
        P.compare_image(out, b, P.oracle_v(cfg, cfg["A"], b, **kw), "bf16", cfg["vis_begin"], False)
