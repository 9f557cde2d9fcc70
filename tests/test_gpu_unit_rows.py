"""Norms, unit rows and column sums of wide bfloat16 features in one pass (decoder calls scored by the mean cosine): rows around a
workgroup's eight and sixteen, features that fill its wavefronts or not, with and without text profiles in the launch.  The unit
rows in the workspace are compared bit for bit, the scores with their definition in float64."""
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


# sequences, system tokens, visual tokens, text tokens, features (16 rows a workgroup from 128 workgroups on)
CASES = [(1, 0, 7, 1, 2048), (1, 3, 8, 33, 2056), (2, 1, 9, 40, 4096), (1, 2, 63, 64, 5120), (1, 5, 65, 31, 8192), (3, 4, 100, 50, 2560),
         (16, 1, 128, 35, 2048), (15, 0, 129, 40, 4104), (128, 2, 15, 3, 2048), (64, 1, 17, 36, 3000), (8, 3, 250, 64, 5120), (127, 0, 16, 2, 2040)]


@pytest.mark.parametrize("B,system,N,M,D", CASES)
def test_unit_rows_and_terms(ctx, B, system, N, M, D):
    g = torch.Generator().manual_seed(N * M + D)
    X = torch.randn(B, system + N + M, D, generator=g) * torch.rand(B, system + N + M, 1, generator=g).add(0.1)
    X[:, system] = 0.0 if N > 8 else X[:, system]                       # a zero row has no direction
    A = torch.softmax(torch.randn(B, 2, M, N, generator=g), -1).to(torch.bfloat16)
    Xd, Ad = X.to(torch.bfloat16).to("cuda"), A.to("cuda")
    p = fc.make_problem(Xd, variant=fc.VARIANT_L, vis_begin=system, N=N, n_keep=max(1, N // 2), w_score=0.6, gamma=0.6, eps=0.998, window=0,
                        red_src=fc.R_SIM_MEAN, sem_src=fc.G_TEXT_ATTN, corr_src=fc.C_COSINE, H=2, A_text=Ad,
                        a_q_begin=system, a_k_begin=system, at_k_begin=system)
    buf = fc.Buffers(p, "cuda", torch.bfloat16)
    buf.ws.fill_(255)
    fc.ficoco_l_step(ctx, p, buf)
    torch.cuda.synchronize()
    x = Xd[:, system:system + N].double()
    n = x.norm(dim=-1, keepdim=True)
    u = torch.where(n > 0, x / n.clamp_min(1e-300), torch.zeros_like(x))
    at = H.gram_plan(p).xhat + buf.ws_ptr - buf.ws.data_ptr()
    got = buf.ws[at:at + B * N * D * 2].view(torch.bfloat16).view(B, N, D)
    # u's double is within 2^-52 of the kernel's: the rounded values can differ where that is a midpoint's distance, which these are not.
    # (torch rounds double to bfloat16 through float: a float that is a midpoint is settled by u itself)
    f = u.float()
    low = f.view(torch.int32) & 0xffff
    mid = low == 0x8000
    up = (u.abs() > f.double().abs()).to(torch.int32)
    ref = torch.where(mid & (u != f.double()), (f.view(torch.int32) - 1 + 2 * up).view(torch.float32), f).to(torch.bfloat16)
    assert torch.equal(got.view(torch.int16), ref.view(torch.int16))
    R = (u @ u.sum(1, keepdim=True).transpose(1, 2))[..., 0] / N
    w = float(torch.tensor(0.6, dtype=torch.float32))
    s = w * R - (1.0 - w) * Ad.double().mean(1).mean(1)
    # sums of at most D + N double terms whose magnitudes add up to one
    assert (buf.scores - s).abs().max().item() <= 4 * (D + N) * 2.0 ** -53 + 1e-13 * s.abs().max().item()
