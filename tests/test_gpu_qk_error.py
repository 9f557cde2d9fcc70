"""Error of the head-mean attention of the [CLS] query against 64 bits, from queries and keys.

Per head a probability carries the roundings of its logit, exponential and normaliser; one head alone shows what they come to
(e1).  Over H heads of like size these average out (e1 / sqrt(H)), and the sum adds one rounding to nearest per partial
sum S_i: within 2^-24 S_i, 2^-24 / sqrt(3) of it rms where the partial sums lie low in their binades.  Sixteen heads in quarters: relative to
the whole sum, squared, four times (1 + 4 + 9 + 16) / 256 and (64 + 144 + 256) / 256, together 2.28 of that; one after the other
1496 / 256 = 5.84.  e1 is taken from three draws, which leaves it uncertain by about a tenth."""
import numpy as np
import pytest
import torch

from paper_2411_17686_amd import ficoco as fc

pytestmark = pytest.mark.gpu


def _cls_error(B, N, H, d, seed):
    g = torch.Generator().manual_seed(seed)
    Q, K = [torch.randn(B, H, N + 1, d, generator=g).to(torch.bfloat16).cuda() for _ in range(2)]
    X = torch.zeros(B, N + 1, 8, dtype=torch.bfloat16, device="cuda")
    ctx = fc.Context(0)
    p = fc.make_problem(X, variant=fc.VARIANT_V, vis_begin=1, N=N, n_keep=N // 2, cls_index=0, window=0, w_score=0.0, Q=Q, K=K)
    buf = fc.Buffers(p, "cuda", X.dtype)
    fc.ficoco_score(ctx, p, buf)
    torch.cuda.synchronize()
    logits = torch.matmul(K.double(), Q[:, :, :1].double().transpose(2, 3).contiguous())[..., 0] * d ** -0.5      # [B][H][N + 1]
    want = -torch.softmax(logits, -1).mean(1)[:, 1:]
    ctx.close()
    return float(((buf.scores - want).pow(2).sum() / want.pow(2).sum()).sqrt())


@pytest.mark.parametrize("B,N,d", [(16, 576, 64), (16, 576, 32), (6, 832, 64)])
def test_cls_row_behind_whole_tiles(B, N, d):
    """65 queries in the last tile of 128: the [CLS] query alone in a wavefront's block."""
    H = 16
    one = np.sqrt(np.mean([_cls_error(B, N, 1, d, s) ** 2 for s in (1, 2, 3)]))
    got = np.sqrt(np.mean([_cls_error(B, N, H, d, s) ** 2 for s in (4, 5, 6)]))
    bound = 1.1 * np.sqrt(one ** 2 / H + 2.28 * (2.0 ** -24 / np.sqrt(3.0)) ** 2)
    assert got <= bound, (one, got, bound)


def _text_error(B, N, H, d, seed):
    """The same of one text query behind N visual ones of a causal map, `system` keys in front of them."""
    g, system = torch.Generator().manual_seed(seed), 3
    n = system + N + 1
    Q, K = [torch.randn(B, H, n, d, generator=g).to(torch.bfloat16).cuda() for _ in range(2)]
    X = torch.zeros(B, n, 8, dtype=torch.bfloat16, device="cuda")
    ctx = fc.Context(0)
    p = fc.make_problem(X, variant=fc.VARIANT_L, vis_begin=system, N=N, n_keep=N // 2, window=0, w_score=0.0, sem_src=fc.G_TEXT_ATTN, Q=Q, K=K, M=1)
    buf = fc.Buffers(p, "cuda", X.dtype)
    fc.ficoco_score(ctx, p, buf)
    torch.cuda.synchronize()
    logits = torch.matmul(K.double(), Q[:, :, -1:].double().transpose(2, 3).contiguous())[..., 0] * d ** -0.5      # [B][H][n]
    want = -torch.softmax(logits, -1).mean(1)[:, system:system + N]
    ctx.close()
    return float(((buf.scores - want).pow(2).sum() / want.pow(2).sum()).sqrt())


@pytest.mark.parametrize("B,N,H", [(4, 512, 32), (8, 384, 32), (5, 512, 16)])
def test_text_row_behind_whole_tiles(B, N, H):
    """Heads of 128, not split, one block of queries in the last tile of 128: four wavefronts share its heads.  Four sums of H / 4 heads, added
    pairwise: squared, relative to the whole sum, 4 (1 + 4 + ... + (H / 4)^2) / H^2 + 2 / 4 + 1 of a rounding's share, 2.3 at 32 heads (11.2 one
    after the other) and 1.97 at sixteen (5.84)."""
    q = H // 4
    shares = 4.0 * q * (q + 1) * (2 * q + 1) / 6 / H ** 2 + 1.5
    one = np.sqrt(np.mean([_text_error(B, N, 1, 128, s) ** 2 for s in (1, 2, 3)]))
    got = np.sqrt(np.mean([_text_error(B, N, H, 128, s) ** 2 for s in (4, 5, 6)]))
    bound = 1.1 * np.sqrt(one ** 2 / H + shares * (2.0 ** -24 / np.sqrt(3.0)) ** 2)
    assert got <= bound, (one, got, bound)
