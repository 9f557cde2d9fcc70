"""Maxima of the text profiles over the visual tokens, read out of the workspace (they only bound a term, so a step's outputs
need not show a wrong one): text queries below, at and above the sixteen of a workgroup, tokens below, at and above a round
of loads (256), formed by the score stage's launch (32 queries or more, fused) or by the correlate stage's."""
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


@pytest.mark.parametrize("visual", [False, True])
@pytest.mark.parametrize("N", [5, 255, 256, 257, 600])
@pytest.mark.parametrize("M", [1, 15, 16, 17, 31, 32, 33, 70])
def test_maxima(ctx, M, N, visual):
    B, D, heads = 3, 32, 2
    g = torch.Generator(device="cuda")
    g.manual_seed(M * 1000 + N)
    X = torch.randn(B, N + M, D, device="cuda", generator=g)
    At = torch.softmax(3.0 * torch.randn(B, heads, M, N, device="cuda", generator=g), -1)
    A = torch.softmax(torch.randn(B, heads, N, N, device="cuda", generator=g), -1) if visual else None
    p = fc.make_problem(X, variant=fc.VARIANT_L, vis_begin=0, N=N, n_keep=max(1, N // 3), A=A, A_text=At, at_k_begin=0, window=0,
                        sem_src=fc.G_TEXT_ATTN, red_src=fc.R_ATTN_RECV if visual else fc.R_SIM_MEAN,
                        corr_src=fc.C_ATTN if visual else fc.C_COSINE)
    want = At.double().mean(1).amax(-1)                     # [B][M]
    plan = H.gram_plan(p)
    for staged in (False, True):
        buf = fc.Buffers(p, "cuda", X.dtype)
        buf.ws.fill_(0xFF)
        if staged:
            fc.ficoco_score(ctx, p, buf)
            fc.ficoco_filter(ctx, p, buf)
            fc.ficoco_correlate(ctx, p, buf)
        else:
            fc.ficoco_l_step(ctx, p, buf)
        torch.cuda.synchronize()
        at = buf.ws_ptr - buf.ws.data_ptr()
        ttext = buf.ws[at + plan.ttext:at + plan.ttext + 8 * B * N * M].view(torch.float64).view(B, N, M)
        cmax = buf.ws[at + plan.cmax:at + plan.cmax + 8 * B * M].view(torch.float64).view(B, M)
        assert torch.equal(cmax, ttext.amax(1)), staged
        assert torch.allclose(cmax, want, rtol=1e-12, atol=0), staged
