"""The block of approximate cosines itself, read out of the workspace, for every form of its tiles.

The block only proposes candidates: whatever it holds, a step decides by exact values, and with small enough values
in it (zeros, say) every target is a candidate and the outputs are right all the same.  So the outputs do not
show a wrong block; here all its values are compared with products of the same unit rows in double precision, within the
error that the readers of the block allow for."""
import pytest
import torch

from paper_2411_17686_amd import ficoco as fc
from tests import plan_hook as H

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = fc.Context(0)
    yield c
    c.close()


def _problem(B, n_disc, n_keep, D, M=0):
    """Unit rows of mixed directions; FiCoCo-L with M text queries, else FiCoCo-V from score vectors."""
    g = torch.Generator(device="cuda")
    g.manual_seed(B + n_disc + n_keep + D + M)
    N = n_disc + n_keep
    X = torch.randn(B, N + M, D, device="cuda", generator=g)
    X += 2.0 * X[:, :1] * torch.rand(B, N + M, 1, device="cuda", generator=g)
    X = X.to(torch.bfloat16)
    if M:
        At = torch.softmax(torch.randn(B, 1, M, N, device="cuda", generator=g), -1).to(torch.bfloat16)
        p = fc.make_problem(X, variant=fc.VARIANT_L, vis_begin=0, N=N, n_keep=n_keep, A_text=At, at_k_begin=0, window=0,
                            sem_src=fc.G_TEXT_ATTN, red_src=fc.R_SIM_MEAN, corr_src=fc.C_COSINE)
        alive = (X, At)
    else:
        v = [torch.softmax(torch.randn(B, 1, N, device="cuda", generator=g), -1).to(torch.bfloat16) for _ in range(2)]
        p = fc.make_problem(X, variant=fc.VARIANT_V, vis_begin=0, N=N, n_keep=n_keep, recv_vec=v[0], sem_vec=v[1], window=0,
                            red_src=fc.R_VECTOR, sem_src=fc.G_VECTOR, corr_src=fc.C_COSINE)
        alive = (X, v)
    buf = fc.Buffers(p, "cuda", X.dtype)
    buf.ws.fill_(0xFF)                      # not-a-numbers wherever the step writes nothing
    return p, buf, alive


def _check(p, buf, plan, S, T):
    """ct[b][a][j] against x[S[b][a]] . x[T[b][j]]; zero where an index is of no token."""
    B, N, nd, nk, D = p.B, p.N, S.shape[1], T.shape[1], plan.Df
    at = buf.ws_ptr - buf.ws.data_ptr()
    ct = buf.ws[at + plan.ct:at + plan.ct + 4 * plan.splits * B * nd * nk].view(torch.float32).view(plan.splits, B, nd, nk)
    xh = buf.ws[at + plan.xhat:at + plan.xhat + 2 * B * N * D].view(torch.bfloat16).view(B, N, D)
    largest = 0.0
    for b0 in range(0, B, 16):
        s, t = S[b0:b0 + 16].long(), T[b0:b0 + 16].long()
        x = xh[b0:b0 + 16].double()

        def rows(i):
            ok = (i >= 0) & (i < N)
            r = torch.gather(x, 1, torch.where(ok, i, 0)[..., None].expand(-1, -1, D))
            return r * ok[..., None]

        want = torch.bmm(rows(s), rows(t).transpose(1, 2).contiguous())
        err = (ct[:, b0:b0 + 16].double().sum(0) - want).abs()
        assert not torch.isnan(err).any(), "values that were not written"
        assert float(err.max()) <= plan.delta, (b0, float(err.max()), plan.delta)
        bad = ((s < 0) | (s >= N))[..., None] | ((t < 0) | (t >= N))[:, None]
        assert (ct[:, b0:b0 + 16].abs().sum(0)[bad] == 0).all()
        largest = max(largest, float(want.abs().max()))
    assert largest > 100 * plan.delta       # a block of zeros would not pass


# images, discarded, kept tokens, features, text queries, form
CASES = [
    # 128 x 128: less than a stage of 32, whole stages, a remainder; several K ranges, the last one shorter
    (3, 127, 129, 8, 0, H.SQUARE), (2, 128, 256, 64, 0, H.SQUARE), (2, 257, 40, 136, 5, H.SQUARE), (1, 300, 200, 1064, 0, H.SQUARE),
    # 192 x 192: seven stages of 64 features (whole turns of the three buffers and what is left), nine, ten, eleven; less than a
    # stage behind them; whole tiles, and rows and columns that miss or pass a tile by one
    (128, 192, 192, 448, 0, H.WIDE), (128, 192, 191, 456, 0, H.WIDE), (128, 193, 191, 480, 0, H.WIDE), (64, 384, 193, 504, 3, H.WIDE),
    (32, 768, 384, 448, 9, H.WIDE), (1, 8064, 1152, 576, 0, H.WIDE), (1, 8000, 1150, 640, 0, H.WIDE), (1, 8060, 1152, 712, 0, H.WIDE),
    # several K ranges: of 512 features; of 544 and 488; of 704 and 648
    (16, 768, 384, 1024, 0, H.WIDE), (16, 760, 383, 1032, 4, H.WIDE), (32, 384, 192, 2056, 0, H.WIDE),
    # 256 x 192: the remainder alone, one stage, two, three and more; whole and edge tiles in one launch
    (150, 256, 192, 24, 0, H.TALL), (64, 500, 193, 72, 6, H.TALL), (86, 512, 384, 64, 0, H.TALL), (64, 512, 200, 200, 0, H.TALL),
    (1, 6216, 3000, 320, 0, H.TALL), (86, 512, 300, 520, 0, H.TALL), (128, 432, 144, 256, 5, H.TALL), (1, 10368, 1152, 136, 0, H.TALL),
    # many tiles of 128 x 128 where larger ones would be mostly padding
    (260, 98, 98, 128, 0, H.SQUARE), (180, 200, 200, 136, 2, H.SQUARE),
]


@pytest.mark.parametrize("B,n_disc,n_keep,D,M,form", CASES)
def test_block_of_every_form(ctx, B, n_disc, n_keep, D, M, form):
    p, buf, alive = _problem(B, n_disc, n_keep, D, M)
    plan = H.gram_plan(p)
    assert plan.use_gram and plan.form == form
    (fc.ficoco_l_step if M else fc.ficoco_v_step)(ctx, p, buf)
    torch.cuda.synchronize()
    _check(p, buf, plan, buf.discard_idx, buf.keep_idx)


@pytest.mark.parametrize("B,n_disc,n_keep,D,M,form", [(2, 200, 150, 72, 0, H.SQUARE), (128, 192, 192, 448, 0, H.WIDE),
                                                      (16, 760, 383, 1032, 4, H.WIDE), (150, 256, 192, 72, 0, H.TALL), (64, 500, 193, 72, 0, H.TALL)])
def test_rows_and_columns_of_no_token_are_zero(ctx, B, n_disc, n_keep, D, M, form):
    """Index sets of the caller (staged calls), some entries outside the image."""
    p, buf, alive = _problem(B, n_disc, n_keep, D, M)
    plan = H.gram_plan(p)
    assert plan.use_gram and plan.form == form
    fc.ficoco_score(ctx, p, buf)
    fc.ficoco_filter(ctx, p, buf)
    for idx in (buf.discard_idx, buf.keep_idx):
        idx[0, 0], idx[0, -1], idx[B - 1, idx.shape[1] // 2], idx[B // 2, 1] = -1, p.N, 2 ** 31 - 1, -2 ** 31
    fc.ficoco_correlate(ctx, p, buf)
    torch.cuda.synchronize()
    _check(p, buf, plan, buf.discard_idx, buf.keep_idx)
    for b, a in ((0, 0), (0, n_disc - 1), (B - 1, n_disc // 2), (B // 2, 1)):
        assert int(buf.edge_cnt[b, a]) == 0


# images, discarded, kept tokens, features, text queries, K ranges: up to 16 tiles of a decoder's layer with long rows are cut into up to
# 16 ranges (the last one shorter, or less than a stage), 17 of them into 8, as the other variant's are
RANGES = [(1, 432, 144, 4096, 64, 16), (1, 128, 128, 4104, 3, 15), (1, 100, 60, 5120, 9, 16), (16, 100, 60, 4096, 2, 16), (17, 100, 60, 4096, 2, 8),
          (1, 129, 129, 2304, 5, 9), (1, 432, 144, 4096, 0, 8)]


@pytest.mark.parametrize("B,n_disc,n_keep,D,M,splits", RANGES)
def test_ranges_of_long_rows(ctx, B, n_disc, n_keep, D, M, splits):
    p, buf, alive = _problem(B, n_disc, n_keep, D, M)
    plan = H.gram_plan(p)
    assert plan.use_gram and plan.form == H.SQUARE and plan.splits == splits
    assert (splits - 1) * plan.st_per_split * 32 < D <= splits * plan.st_per_split * 32
    (fc.ficoco_l_step if M else fc.ficoco_v_step)(ctx, p, buf)
    torch.cuda.synchronize()
    _check(p, buf, plan, buf.discard_idx, buf.keep_idx)
