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


def _problem(Xd, Ad, system, N, F=None):
    return fc.make_problem(Xd, variant=fc.VARIANT_L, vis_begin=system, N=N, n_keep=max(1, N // 2), w_score=0.6, gamma=0.6, eps=0.998, window=0,
                           red_src=fc.R_SIM_MEAN, sem_src=fc.G_TEXT_ATTN, corr_src=fc.C_COSINE, H=2, A_text=Ad, F=F,
                           a_q_begin=system, a_k_begin=system, at_k_begin=system)


def _unit_rows(p, buf):
    at = H.gram_plan(p).xhat + buf.ws_ptr - buf.ws.data_ptr()
    return buf.ws[at:at + p.B * p.N * H.gram_plan(p).Df * 2].view(torch.bfloat16).view(p.B, p.N, -1)


# sequences, visual tokens, text tokens, features, room behind a row and behind a sequence (odd: rows at any 2-byte address)
STRIDES = [(1, 40, 5, 2048, 1, 0), (3, 65, 40, 2056, 7, 3), (2, 129, 33, 4096, 8, 1), (16, 131, 36, 5120, 3, 2), (2, 33, 64, 8192, 5, 0)]


@pytest.mark.parametrize("separate", [False, True])
@pytest.mark.parametrize("B,N,M,D,room,behind", STRIDES)
def test_rows_with_room_behind_them(ctx, B, N, M, D, room, behind, separate):
    """The same bits from rows and sequences apart in memory, with NaN between, as from contiguous ones; as tokens and as features of their own."""
    assert (B * ((N + 15) // 16) >= 128) == (B == 16)          # both numbers of rows a workgroup
    system, n = 3, 3 + N + M
    g = torch.Generator().manual_seed(N + D)
    X = torch.randn(B, n, D, generator=g).to(torch.bfloat16).to("cuda")
    A = torch.softmax(torch.randn(B, 2, M, N, generator=g), -1).to(torch.bfloat16).to("cuda")
    flat = torch.full((B * (n * (D + room) + behind) + 1,), float("nan"), dtype=torch.bfloat16, device="cuda")
    apart = flat.as_strided((B, n, D), (n * (D + room) + behind, D + room, 1), 1 if room % 2 else 0)
    apart.copy_(X)
    tokens = torch.randn(B, n, 64, generator=g).to(torch.bfloat16).to("cuda")
    outs = []
    for f in (X, apart):
        p = _problem(tokens, A, system, N, F=f[:, system:system + N]) if separate else _problem(f, A, system, N)
        assert p.D >= 2048 or p.Df >= 2048
        buf = fc.Buffers(p, "cuda", torch.bfloat16)
        buf.ws.fill_(255)
        fc.ficoco_l_step(ctx, p, buf)
        torch.cuda.synchronize()
        outs.append([_unit_rows(p, buf).clone().view(torch.int16)] + [getattr(buf, k) for k in ("scores", "keep_idx", "edge_cnt", "X_out")])
    for a, b in zip(*outs):
        assert torch.equal(a, b)


@pytest.mark.parametrize("D,N", [(2048, 20), (4104, 65)])
def test_infinities_and_nan_stay_in_their_sequence(ctx, D, N):
    """A row with an infinity has no direction but where it is infinite, one with NaN none at all: zeros and NaN there, and every other
    sequence's rows and scores as without them."""
    B, M, system = 3, 40, 2
    g = torch.Generator().manual_seed(D)
    X = torch.randn(B, system + N + M, D, generator=g).to(torch.bfloat16)
    A = torch.softmax(torch.randn(B, 2, M, N, generator=g), -1).to(torch.bfloat16).to("cuda")
    bad = X.clone()
    bad[1, system + 3, 5], bad[1, system + 3, D - 1] = float("inf"), float("-inf")
    bad[1, system + N - 1, 0] = float("nan")
    got = []
    for x in (X, bad):
        xd = x.to("cuda")
        p = _problem(xd, A, system, N)
        buf = fc.Buffers(p, "cuda", torch.bfloat16)
        fc.ficoco_score(ctx, p, buf)
        torch.cuda.synchronize()
        got.append((_unit_rows(p, buf).clone(), buf.scores.clone()))
    (u, s), (ub, sb) = got
    for b in (0, 2):
        assert torch.equal(u[b].view(torch.int16), ub[b].view(torch.int16)) and torch.equal(s[b], sb[b])
    # the mean unit row has the NaN, and with it every product but that of the row whose norm is no number: like a zero row it has no cosine
    assert torch.isnan(sb[1, :N - 1]).all() and torch.isfinite(sb[1, N - 1])
    nan = torch.zeros(N, D, dtype=torch.bool)
    nan[3, 5] = nan[3, D - 1] = nan[N - 1, 0] = True
    assert torch.equal(torch.isnan(ub[1]).cpu(), nan)
    rows = [3, N - 1]
    assert bool((ub[1][rows][~nan[rows].to("cuda")] == 0).all())
    keep = [i for i in range(N) if i not in rows]
    assert torch.equal(ub[1][keep].view(torch.int16), u[1][keep].view(torch.int16))
