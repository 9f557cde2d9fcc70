"""The step fed with projected queries and keys instead of the attention maps (Sec.
"Self-Attention", A = Softmax(Q K^T / sqrt(D))): the library forms the per-head softmax on the
matrix cores in single precision and never stores [B,H,n,n]; the oracle forms it in float64.

Bar.  Scores and map entries agree to about 1e-6, not to the last bit, so the comparison is the
margin rule: every top-K decision and every threshold decision whose relative margin (from the
oracle's float64 values) exceeds 64 * 2^-24 must be identical; where all decisions of an image are
identical, weights and merged tokens must agree within the token tolerance (bfloat16: 2e-2
relative / 1e-2 absolute; float32: 1e-5 of the row's largest magnitude)."""
import sys

import numpy as np
import pytest
import torch

from oracle import ficoco_oracle as O
from paper_2411_17686_amd import ficoco as fc
from paper_2411_17686_amd import synth
from tests import parity as P

pytestmark = pytest.mark.gpu


def say(msg):
    print(msg, file=sys.stderr, flush=True)


def draw_qk(seed, B, H, n, d, sigma):
    """Queries and keys whose logits q.k / sqrt(d) are about N(0, sigma^2), as bfloat16."""
    g = torch.Generator().manual_seed(seed)
    Q = (torch.randn(B, H, n, d, generator=g) * sigma ** 0.5).to(torch.bfloat16)
    K = (torch.randn(B, H, n, d, generator=g) * sigma ** 0.5).to(torch.bfloat16)
    return Q, K


def run_qk(ctx, cfg, Q, K, **kw):
    Xd, Qd, Kd = cfg["X"].to("cuda"), Q.to("cuda"), K.to("cuda")
    p = fc.make_problem(Xd, variant=fc.VARIANT_V, vis_begin=cfg["vis_begin"], N=cfg["N"], n_keep=cfg["n_keep"],
                        cls_index=cfg["cls_index"], grid=cfg["grid"], window=cfg["window"], penalty_coef=cfg["coef"],
                        w_score=cfg["lam"], eps=cfg["eps"], Q=Qd, K=Kd, qk_begin=0, **kw)
    buf = fc.Buffers(p, "cuda", Xd.dtype)
    fc.ficoco_v_step(ctx, p, buf)
    out = P.gpu_outputs(buf)
    del Xd, Qd, Kd
    return out


def compare_under_margin_rule(out, b, ref, dtype, vis_begin):
    """Returns True when every decision of the image agreed (then the values were compared too)."""
    scale = float(np.max(np.abs(ref["scores"])))
    assert np.all(np.abs(out["scores"][b] - ref["scores"]) <= 8e-6 * scale), "scores beyond single-precision accuracy"
    same_sets = np.array_equal(out["discard"][b], ref["S"])
    if not same_sets:
        # only decisions inside the margin may differ: checked token by token
        P.margin_audit(dict(out, cnt=np.zeros_like(out["cnt"])), b, dict(ref, tau=None))
        return False
    P.margin_audit(out, b, ref)
    same_J = all(out["cnt"][b, a] == len(J) and np.array_equal(out["tgt"][b, a, :len(J)], J)
                 for a, J in enumerate(ref["J"]))
    if not same_J:
        return False
    for a, J in enumerate(ref["J"]):
        np.testing.assert_allclose(out["alpha"][b, a, :len(J)], ref["alpha"][a], rtol=2e-5)
    got, want = O.widen(out["X_out"][b]), ref["X_out"]
    err = np.abs(got - want)
    if dtype == "f32":
        assert np.all(err <= 1e-5 * np.max(np.abs(want), axis=1, keepdims=True))
    else:
        assert np.all(err <= 2e-2 * np.abs(want) + 1e-2)
    if ref["pos_out"] is not None:
        assert np.array_equal(out["pos_out"][b], ref["pos_out"])
    return True


@pytest.fixture(scope="module")
def ctx():
    c = fc.Context(0)
    yield c
    c.close()


def _case(ctx, seed, B, grid, D, H, d, dtype, n_keep, sigma):
    cfg = synth.ficoco_v_single(seed=seed, B=B, grid=grid, D=D, H=1, centres=8, dtype=dtype, n_keep=n_keep)
    Q, K = draw_qk(seed + 1, B, H, cfg["N"] + 1, d, sigma)
    out = run_qk(ctx, cfg, Q, K)
    full = 0
    for b in range(B):
        ref = O.v_step_qk(O.widen(synth.to_numpy(cfg["X"][b])), O.widen(synth.to_numpy(Q[b])), O.widen(synth.to_numpy(K[b])),
                          float(d) ** -0.5, cls_index=0, vis_begin=1, N=cfg["N"], n_keep=n_keep, lam=cfg["lam"],
                          eps=cfg["eps"], grid=cfg["grid"], window=2, coef=2.0)
        full += compare_under_margin_rule(out, b, ref, dtype, 1)
    return full


def test_config0_shape_from_queries_and_keys(ctx):
    full = _case(ctx, 40, 1, 24, 1024, 16, 64, "f32", 192, 1.0)
    say("config 0 shape from Q, K: %d of 1 images with every decision identical" % full)


def test_config1_shape_from_queries_and_keys(ctx):
    full = _case(ctx, 41, 16, 24, 1024, 16, 64, "bf16", 384, 1.5)
    say("config 1 shape from Q, K: %d of 16 images with every decision identical" % full)
    assert full >= 12          # in-margin decisions are rare


@pytest.mark.parametrize("seed,grid,H,d,n_keep", [(1, 7, 3, 32, 20), (2, 16, 5, 32, 100), (3, 19, 2, 128, 301), (4, 25, 4, 64, 625),
                                                  (5, 5, 1, 64, 1)])
def test_small_and_ragged_shapes(ctx, seed, grid, H, d, n_keep):
    full = _case(ctx, 50 + seed, 2, grid, 72, H, d, ["f32", "bf16"][seed % 2], n_keep, 1.0)
    assert full >= 1


def test_long_sequence_at_full_width_from_queries_and_keys(ctx):
    """2304 patches + [CLS], 16 heads of 64, D = 1024, 640 preserved."""
    full = _case(ctx, 42, 2, 48, 1024, 16, 64, "bf16", 640, 1.0)
    say("2304-patch shape from Q, K: %d of 2 images with every decision identical" % full)


@pytest.mark.parametrize("seed,grid,H,d,n_keep", [(1, 27, 3, 64, 300), (2, 36, 2, 32, 500), (3, 31, 5, 128, 700),
                                                  (4, 40, 1, 64, 1000)])
def test_sequences_longer_than_one_key_block(ctx, seed, grid, H, d, n_keep):
    """730, 1297, 962 and 1601 keys with one to five heads: more keys than heads are unlimited for."""
    full = _case(ctx, 70 + seed, 2, grid, 72, H, d, ["f32", "bf16"][seed % 2], n_keep, 1.0)
    assert full >= 1


def _case_l(ctx, seed, B, n_sys, N, M, D, H, d, n_keep, red, corr, sigma=1.0, staged=False):
    """FiCoCo-L fed the decoder layer's queries and keys (causal maps; the text tokens follow the
    visual span) against the oracle's float64 evaluation, under the margin rule."""
    cfg = synth.ficoco_l_decoder(seed=seed, B=B, n_sys=n_sys, N=N, M=M, D=D, H=1, centres=8, n_keep=n_keep, with_vv=False)
    n_tot = n_sys + N + M
    Q, K = draw_qk(seed + 1, B, H, n_tot, d, sigma)
    Xd, Qd, Kd = cfg["X"].to("cuda"), Q.to("cuda"), K.to("cuda")
    p = fc.make_problem(Xd, variant=fc.VARIANT_L, vis_begin=n_sys, N=N, n_keep=n_keep, w_score=cfg["beta"],
                        gamma=cfg["gamma"], eps=cfg["eps"], red_src=red, sem_src=fc.G_TEXT_ATTN, corr_src=corr,
                        window=0, Q=Qd, K=Kd, qk_begin=0, M=M)
    buf = fc.Buffers(p, "cuda", Xd.dtype)
    if staged:
        fc.ficoco_score(ctx, p, buf)
        fc.ficoco_filter(ctx, p, buf)
        fc.ficoco_correlate(ctx, p, buf)
        fc.ficoco_compress(ctx, p, buf)
    else:
        fc.ficoco_l_step(ctx, p, buf)
    out = P.gpu_outputs(buf)
    del Xd, Qd, Kd
    full = 0
    names = {fc.R_ATTN_RECV: "attn", fc.R_SIM_MEAN: "sim_mean", fc.C_ATTN: "attn", fc.C_COSINE: "cosine"}
    for b in range(B):
        ref = O.l_step_qk(O.widen(synth.to_numpy(cfg["X"][b])), O.widen(synth.to_numpy(Q[b])), O.widen(synth.to_numpy(K[b])),
                          float(d) ** -0.5, vis_begin=n_sys, N=N, M=M, n_keep=n_keep, beta=cfg["beta"], gamma=cfg["gamma"],
                          eps=cfg["eps"], red_src=names[red], corr_src="attn" if corr == fc.C_ATTN else "cosine")
        full += compare_under_margin_rule(out, b, ref, cfg["dtype"], n_sys)
    return full


@pytest.mark.parametrize("red,corr", [(fc.R_ATTN_RECV, fc.C_ATTN), (fc.R_SIM_MEAN, fc.C_COSINE), (fc.R_ATTN_RECV, fc.C_COSINE)])
@pytest.mark.parametrize("shape", [(3, 77, 9, 72, 3, 32, 31), (35, 576, 64, 128, 4, 64, 144), (5, 1300, 40, 72, 2, 128, 700),
                                   (0, 100, 1, 64, 1, 64, 50)])
def test_decoder_step_from_queries_and_keys(ctx, shape, red, corr):
    """89, 675, 1345 and 101 positions; with the visual-to-visual terms (tiles over the visual and the text queries) and without (text queries
    alone); 1 to 64 text queries."""
    n_sys, N, M, D, H, d, n_keep = shape
    full = _case_l(ctx, 80 + N % 50, 2, n_sys, N, M, D, H, d, n_keep, red, corr)
    assert full >= 1


@pytest.mark.parametrize("red,corr", [(fc.R_ATTN_RECV, fc.C_ATTN), (fc.R_SIM_MEAN, fc.C_COSINE)])
def test_decoder_stages_from_queries_and_keys(ctx, red, corr):
    """The same through the staged entry points (score, filter, correlate, compress one call each)."""
    assert _case_l(ctx, 91, 2, 4, 130, 33, 72, 6, 64, 60, red, corr, staged=True) >= 1


def test_unsupported_shapes_are_refused(ctx):
    cfg = synth.ficoco_v_single(seed=9, B=1, grid=4, D=8, H=1, centres=2, dtype="bf16", n_keep=8)
    Xd = cfg["X"].to("cuda")
    for n, d in ((17, 24), (17, 16), (17, 256)):
        Q = torch.zeros(1, 2, n, d, dtype=torch.bfloat16, device="cuda")
        p = fc.make_problem(Xd, variant=fc.VARIANT_V, vis_begin=1, N=16, n_keep=8, cls_index=0, grid=(1, 4, 4), window=2,
                            Q=Q, K=Q.clone())
        with pytest.raises(fc.FicocoError) as e:
            fc.workspace_bytes(p)
        assert e.value.code == fc.EUNSUPPORTED
    # beyond 640 rows: at most 64 heads
    cfg = synth.ficoco_v_single(seed=9, B=1, grid=26, D=8, H=1, centres=2, dtype="bf16", n_keep=8)
    Xd = cfg["X"].to("cuda")
    Q = torch.zeros(1, 65, 677, 32, dtype=torch.bfloat16, device="cuda")
    p = fc.make_problem(Xd, variant=fc.VARIANT_V, vis_begin=1, N=676, n_keep=8, cls_index=0, grid=(1, 26, 26), window=2,
                        Q=Q, K=Q.clone())
    with pytest.raises(fc.FicocoError) as e:
        fc.workspace_bytes(p)
    assert e.value.code == fc.EUNSUPPORTED


@pytest.mark.parametrize("B,grid,H,d", [(1, 3, 2, 64), (2, 4, 9, 32), (1, 12, 3, 128), (2, 12, 8, 64), (16, 24, 3, 32), (40, 10, 2, 64),
                                        (3, 21, 5, 128)])
def test_query_tiles_and_head_shares(ctx, B, grid, H, d):
    """Edges of the two kernels' tiles (48 query rows of the row normalisers, 64 or 128 of the head mean, 64 keys): one block of
    queries in all, the [CLS] query alone behind whole tiles; few tiles (heads split over four groups of
    wavefronts from eight heads on: 9 in shares of three, the last one without any, and 8) and many (not)."""
    full = _case(ctx, 300 + B + grid, B, grid, 72, H, d, "bf16", max(1, grid * grid // 3), 1.0)
    assert full >= (B + 1) // 2


@pytest.mark.parametrize("B,grid,H,d", [(1, 8, 5, 64), (1, 9, 6, 128), (63, 9, 3, 64), (64, 9, 2, 128), (50, 16, 2, 64), (6, 18, 17, 128),
                                        (70, 10, 3, 32)])
def test_tiles_of_64_and_128_queries_of_the_head_mean(ctx, B, grid, H, d):
    """65 queries (a block of a wide tile and one query more), 82 (18 more), 257 (two wide tiles and one query left) and 101 (a wide
    tile that is not full); 325 with 17 heads in tiles of 64, split (108 workgroups), of which 5 queries are left."""
    full = _case(ctx, 360 + B + grid, B, grid, 72, H, d, "bf16", max(1, grid * grid // 3), 1.0)
    assert full >= (B + 1) // 2


@pytest.mark.parametrize("B,N,M,H,d", [(30, 230, 40, 2, 64), (1, 230, 40, 6, 128), (40, 100, 33, 3, 32)])
def test_causal_tiles_of_64_and_128_queries(ctx, B, N, M, H, d):
    """270 queries of which a block of 14 is left behind wide tiles, few heads on few tiles, and 133."""
    full = _case_l(ctx, 380 + B, B, 3, N, M, 72, H, d, N // 3, fc.R_ATTN_RECV, fc.C_ATTN)
    assert full >= (B + 1) // 2


@pytest.mark.parametrize("B,grid,H,d", [(16, 24, 3, 64), (16, 24, 4, 64), (16, 14, 15, 32), (32, 14, 16, 32)])
def test_keys_shared_by_the_wavefronts_or_not(ctx, B, grid, H, d):
    """192 and 256 workgroups of the row normalisers with heads of 64, 480 and 1024 with heads of 32: below 256
    and 640 the wavefronts of a workgroup share the keys of a query tile."""
    full = _case(ctx, 330 + B + H, B, grid, 72, H, d, "bf16", grid * grid // 3, 1.0)
    assert full >= (B + 1) // 2


@pytest.mark.parametrize("B,grid,H,d", [(16, 14, 5, 128), (16, 14, 6, 128), (13, 14, 24, 32), (20, 14, 16, 32)])
def test_keys_shared_at_the_other_head_sizes(ctx, B, grid, H, d):
    """160 and 192 workgroups with heads of 128 (shared below 192), 624 and 640 with heads of 32 (below 640)."""
    full = _case(ctx, 350 + B + H, B, grid, 72, H, d, "bf16", grid * grid // 3, 1.0)
    assert full >= (B + 1) // 2


@pytest.mark.parametrize("B,grid,H,d", [(1, 8, 7, 64), (1, 8, 8, 64), (1, 8, 9, 64), (1, 9, 10, 128), (1, 16, 11, 64), (2, 10, 13, 32), (8, 18, 17, 128)])
def test_heads_split_from_eight_on(ctx, B, grid, H, d):
    """Few tiles: seven heads together, eight and more in four shares of two to four, the last one empty (9) or shorter (10, 11, 13);
    65, 82, 257 and 101 queries in tiles of 64 (one, 18, one and 37 left); 144 workgroups (not split)."""
    full = _case(ctx, 390 + B + H, B, grid, 72, H, d, "bf16", max(1, grid * grid // 3), 1.0)
    assert full >= (B + 1) // 2


@pytest.mark.parametrize("B,N,M,H,d", [(1, 230, 40, 9, 128), (2, 100, 33, 8, 32), (1, 61, 40, 13, 64)])
def test_causal_heads_split(ctx, B, N, M, H, d):
    """270 queries in tiles of 64 (a block of 14 left), 133 (5 left) and 101 (37 left), heads in shares."""
    full = _case_l(ctx, 400 + B + H, B, 3, N, M, 72, H, d, N // 3, fc.R_ATTN_RECV, fc.C_ATTN)
    assert full >= (B + 1) // 2


@pytest.mark.parametrize("B,N,M,H", [(1, 70, 5, 1), (2, 64, 64, 2), (1, 130, 33, 3), (2, 200, 9, 4), (1, 129, 128, 5), (1, 61, 70, 6), (3, 128, 1, 7),
                                     (1, 193, 64, 12), (2, 33, 31, 13), (9, 250, 40, 17), (11, 250, 40, 12), (22, 130, 33, 17), (1, 20, 20, 18)])
def test_causal_heads_of_128(ctx, monkeypatch, B, N, M, H):
    """Heads that leave every remainder of a turn of six; one tile, tiles of zeros, tiles with one wavefront's queries; eight heads and
    more with 132 tiles, and with fewer (split, not that form).  The workspace holds NaN first: every entry of the maps has to be written."""
    make = fc.Buffers

    def filled(*args):
        buf = make(*args)
        buf.ws.fill_(255)
        return buf
    monkeypatch.setattr(fc, "Buffers", filled)
    full = _case_l(ctx, 440 + B + H + N, B, 3, N, M, 72, H, 128, max(1, N // 3), fc.R_ATTN_RECV, fc.C_ATTN)
    assert full >= (B + 1) // 2


@pytest.mark.parametrize("B,N,M,H,d", [(16, 64, 200, 16, 64), (13, 50, 200, 13, 64), (8, 64, 200, 25, 128), (7, 30, 400, 31, 128), (5, 500, 60, 21, 64)])
def test_causal_normalisers_head_by_head_or_long_first(ctx, B, N, M, H, d):
    """Two groups of queries that see about the same keys (head by head), three and four (long first, a number of heads that does not divide among
    the XCDs)."""
    full = _case_l(ctx, 470 + B + H, B, 3, N, M, 72, H, d, N // 3, fc.R_ATTN_RECV, fc.C_ATTN)
    assert full >= (B + 1) // 2


def _same_bits(ctx, kw, Q, K, X):
    """One step from contiguous queries and keys, and from the same ones as a projection leaves them ([B][n][H][d], with room behind a row)."""
    B, H, n, d = Q.shape
    outs = []
    for apart in (False, True):
        q, k = Q.to("cuda"), K.to("cuda")
        if apart:
            both = torch.full((B, n, 2 * H * d + 8), float("nan"), dtype=torch.bfloat16, device="cuda")
            at_q, at_k = both[..., :H * d].unflatten(-1, (H, d)), both[..., H * d:2 * H * d].unflatten(-1, (H, d))
            at_q.copy_(q.transpose(1, 2))
            at_k.copy_(k.transpose(1, 2))
            q, k = at_q.transpose(1, 2), at_k.transpose(1, 2)
        p = fc.make_problem(X, Q=q, K=k, qk_begin=0, **kw)
        assert not apart or (p.qk_stride_h, p.qk_stride_n) == (d, 2 * H * d + 8)
        buf = fc.Buffers(p, "cuda", X.dtype)
        buf.ws.fill_(255)
        (fc.ficoco_l_step if kw["variant"] == fc.VARIANT_L else fc.ficoco_v_step)(ctx, p, buf)
        torch.cuda.synchronize()
        outs.append([getattr(buf, name) for name in ("scores", "keep_idx", "edge_cnt", "X_out")])
    for a, b in zip(*outs):
        assert torch.equal(a, b)


@pytest.mark.parametrize("B,N,M,H,d", [(1, 130, 33, 3, 128), (5, 600, 60, 7, 128), (2, 129, 70, 17, 128), (3, 200, 20, 13, 64), (2, 90, 150, 8, 32), (1, 60, 17, 32, 128),
                                       (16, 64, 200, 16, 64)])
def test_causal_queries_and_keys_as_a_projection_leaves_them(ctx, B, N, M, H, d):
    """Heads of 128 in whole tiles (of 163 and 660 queries: 300 tiles, live ones first, a whole turn of six heads and one more), split, text queries
    shared by wavefronts, normalisers long first and head by head."""
    g = torch.Generator().manual_seed(B + N + H)
    n = 3 + N + M
    Q, K = draw_qk(B + N + H, B, H, n, d, 1.0)
    X = torch.randn(B, n, 72, generator=g).to(torch.bfloat16).to("cuda")
    _same_bits(ctx, dict(variant=fc.VARIANT_L, vis_begin=3, N=N, n_keep=max(1, N // 3), w_score=0.6, gamma=0.6, eps=0.998, window=0, M=M,
                         red_src=fc.R_ATTN_RECV, sem_src=fc.G_TEXT_ATTN, corr_src=fc.C_ATTN), Q, K, X)


@pytest.mark.parametrize("B,N,H,d", [(1, 64, 3, 64), (16, 196, 9, 32), (2, 289, 8, 64), (3, 400, 17, 128)])
def test_queries_and_keys_as_a_projection_leaves_them(ctx, B, N, H, d):
    g = torch.Generator().manual_seed(B + N + H)
    Q, K = draw_qk(B + N + H + 1, B, H, N + 1, d, 1.0)
    X = torch.randn(B, N + 1, 72, generator=g).to(torch.bfloat16).to("cuda")
    _same_bits(ctx, dict(variant=fc.VARIANT_V, vis_begin=1, N=N, n_keep=N // 2, cls_index=0, window=0, eps=0.998), Q, K, X)


@pytest.mark.parametrize("M,H,d", [(1, 32, 128), (16, 16, 128), (17, 9, 128), (32, 32, 64), (31, 17, 64), (32, 16, 64), (5, 64, 32), (33, 40, 32)])
def test_one_block_of_text_queries(ctx, M, H, d):
    """At most 32 text queries alone, heads split: by wavefronts that share the heads, or (four 32-feature steps a wavefront and
    more) as any other tile; one query more."""
    full = _case_l(ctx, 420 + M + H, 2, 5, 90, M, 72, H, d, 30, fc.R_SIM_MEAN, fc.C_COSINE)
    assert full >= 1


@pytest.mark.parametrize("grid,H,d,where", [(24, 2, 64, 500), (24, 2, 64, 40), (12, 3, 32, 144), (30, 1, 128, 33), (3, 2, 64, 9)])
def test_logits_far_above_those_of_the_first_keys(ctx, grid, H, d, where):
    """Rows whose largest logit lies 100 to 300 (units of e) above those of the keys the softmax
    reference is taken from: nearly all attention goes to that key, on queries of either sign."""
    cfg = synth.ficoco_v_single(seed=77, B=1, grid=grid, D=72, H=1, centres=8, dtype="bf16", n_keep=grid * grid // 2)
    Q, K = draw_qk(78, 1, H, cfg["N"] + 1, d, 1.0)
    K[:, :, where] = (K[:, :, where].float() * 40.0).to(torch.bfloat16)
    Q = (Q.float() * 8.0).to(torch.bfloat16)
    out = run_qk(ctx, cfg, Q, K)
    ref = O.v_step_qk(O.widen(synth.to_numpy(cfg["X"][0])), O.widen(synth.to_numpy(Q[0])), O.widen(synth.to_numpy(K[0])),
                      float(d) ** -0.5, cls_index=0, vis_begin=1, N=cfg["N"], n_keep=cfg["n_keep"], lam=cfg["lam"],
                      eps=cfg["eps"], grid=cfg["grid"], window=2, coef=2.0)
    # logits up to a few hundred are rounded to 2^-24 of themselves in single precision: probabilities to about 3e-5
    assert np.all(np.isfinite(out["scores"][0]))
    assert np.max(np.abs(out["scores"][0] - ref["scores"])) <= 6e-5 * np.max(np.abs(ref["scores"]))


def test_images_in_rounds(ctx):
    """More images than the row normalisers have room for at a time (40 x 64 heads x 577 queries: two rounds of
    20): scores, edges, weights and tokens on both sides of the border."""
    B, grid, H, d = 40, 24, 64, 32
    cfg = synth.ficoco_v_single(seed=5, B=B, grid=grid, D=8, H=1, centres=8, dtype="bf16", n_keep=100)
    Q, K = draw_qk(6, B, H, cfg["N"] + 1, d, 1.0)
    out = run_qk(ctx, cfg, Q, K)
    full = 0
    for b in (0, 19, 20, 39):
        ref = O.v_step_qk(O.widen(synth.to_numpy(cfg["X"][b])), O.widen(synth.to_numpy(Q[b])), O.widen(synth.to_numpy(K[b])),
                          float(d) ** -0.5, cls_index=0, vis_begin=1, N=cfg["N"], n_keep=100, lam=cfg["lam"],
                          eps=cfg["eps"], grid=cfg["grid"], window=2, coef=2.0)
        full += compare_under_margin_rule(out, b, ref, "bf16", 1)
    assert full >= 3


@pytest.mark.parametrize("B,N,M,red,corr,check", [
    (130, 100, 40, fc.R_ATTN_RECV, fc.C_ATTN, (0, 64, 65, 129)),         # 140 queries of 64 heads: two rounds of 65
    (560, 40, 30, fc.R_SIM_MEAN, fc.C_COSINE, (0, 279, 280, 559)),       # the text queries alone: two rounds of 280
    (3, 60, 21, fc.R_ATTN_RECV, fc.C_ATTN, (0, 1, 2)),
])
def test_decoder_images_in_rounds_and_rows_beyond_the_text(ctx, B, N, M, red, corr, check):
    """The causal form in rounds of images, with rows behind the text tokens that are no query of the step."""
    n_sys, tail, H, d, D, n_keep = 3, 19, 64, 32, 16, N // 3
    cfg = synth.ficoco_l_decoder(seed=15, B=B, n_sys=n_sys, N=N, M=M + tail, D=D, H=1, centres=8, n_keep=n_keep, with_vv=False)
    Q, K = draw_qk(16, B, H, n_sys + N + M + tail, d, 1.0)
    Q[:, :, n_sys + N + M:] = 100.0                          # (a query from there would be seen)
    K[:, :, n_sys + N + M:] = 100.0
    Xd, Qd, Kd = cfg["X"].to("cuda"), Q.to("cuda"), K.to("cuda")
    p = fc.make_problem(Xd, variant=fc.VARIANT_L, vis_begin=n_sys, N=N, n_keep=n_keep, w_score=cfg["beta"],
                        gamma=cfg["gamma"], eps=cfg["eps"], red_src=red, sem_src=fc.G_TEXT_ATTN, corr_src=corr,
                        window=0, Q=Qd, K=Kd, qk_begin=0, M=M)
    buf = fc.Buffers(p, "cuda", Xd.dtype)
    fc.ficoco_l_step(ctx, p, buf)
    out = P.gpu_outputs(buf)
    del Xd, Qd, Kd
    full = 0
    for b in check:
        ref = O.l_step_qk(O.widen(synth.to_numpy(cfg["X"][b])), O.widen(synth.to_numpy(Q[b])), O.widen(synth.to_numpy(K[b])),
                          float(d) ** -0.5, vis_begin=n_sys, N=N, M=M, n_keep=n_keep, beta=cfg["beta"], gamma=cfg["gamma"],
                          eps=cfg["eps"], red_src="attn" if red == fc.R_ATTN_RECV else "sim_mean",
                          corr_src="attn" if corr == fc.C_ATTN else "cosine")
        full += compare_under_margin_rule(out, b, ref, cfg["dtype"], n_sys)
    assert full >= len(check) - 1


@pytest.mark.parametrize("B,N,M,H,d,visual", [(1, 300, 7, 3, 64, False), (1, 260, 16, 3, 32, False), (1, 300, 17, 3, 64, False),
                                              (1, 150, 60, 3, 128, True), (2, 290, 60, 64, 64, True)])
def test_causal_logits_far_above_those_of_the_first_keys(ctx, B, N, M, H, d, visual):
    """The decoder's causal form where a visual and a text key lie far above the first 32: rows that are done again
    with their own maximum, and, for queries before such a key, probabilities beyond single precision that must not
    be seen.  16 queries or fewer, one tile whose keys the wavefronts share, and whole tiles per wavefront (the
    last).  Logits of a few hundred are rounded to 2^-24 of themselves: probabilities to about 3e-5, so decisions
    are compared where the margin exceeds 1e-3."""
    n_sys, D, n_keep = 4, 72, N // 3
    cfg = synth.ficoco_l_decoder(seed=83, B=B, n_sys=n_sys, N=N, M=M, D=D, H=1, centres=8, n_keep=n_keep, with_vv=False)
    Q, K = draw_qk(84, B, H, n_sys + N + M, d, 1.0)
    for where in (n_sys + N - 20, n_sys + N + M // 2):
        K[:, :, where] = (K[:, :, where].float() * 40.0).to(torch.bfloat16)
    Q = (Q.float() * 8.0).to(torch.bfloat16)
    x = (Q[0].float() @ K[0].float().transpose(1, 2)) * float(d) ** -0.5
    first = torch.stack([x[:, n_sys + N:, c:c + 32].amax(2) for c in (0, 32, 64, 96)]).amin(0)
    assert (x[:, n_sys + N:, n_sys + N - 20] - first).max() > 90     # (beyond 2^100 relative to any wavefront's reference)
    Xd, Qd, Kd = cfg["X"].to("cuda"), Q.to("cuda"), K.to("cuda")
    p = fc.make_problem(Xd, variant=fc.VARIANT_L, vis_begin=n_sys, N=N, n_keep=n_keep, w_score=cfg["beta"],
                        gamma=cfg["gamma"], eps=cfg["eps"], red_src=fc.R_ATTN_RECV if visual else fc.R_SIM_MEAN,
                        sem_src=fc.G_TEXT_ATTN, corr_src=fc.C_ATTN if visual else fc.C_COSINE, window=0, Q=Qd, K=Kd, qk_begin=0, M=M)
    buf = fc.Buffers(p, "cuda", Xd.dtype)
    fc.ficoco_l_step(ctx, p, buf)
    out = P.gpu_outputs(buf)
    del Xd, Qd, Kd
    ref = O.l_step_qk(O.widen(synth.to_numpy(cfg["X"][0])), O.widen(synth.to_numpy(Q[0])), O.widen(synth.to_numpy(K[0])),
                      float(d) ** -0.5, vis_begin=n_sys, N=N, M=M, n_keep=n_keep, beta=cfg["beta"], gamma=cfg["gamma"],
                      eps=cfg["eps"], red_src="attn" if visual else "sim_mean", corr_src="attn" if visual else "cosine")
    scale = np.max(np.abs(ref["scores"]))
    assert np.max(np.abs(out["scores"][0] - ref["scores"])) <= 6e-5 * scale
    assert np.all(np.isfinite(O.widen(out["X_out"][0])))
    order = np.sort(ref["scores"])[::-1]
    cut = 0.5 * (order[N - n_keep - 1] + order[N - n_keep])
    far = np.abs(ref["scores"] - cut) > 1e-3 * scale
    gone = np.zeros(N, bool)
    gone[out["discard"][0]] = True
    assert np.array_equal(gone[far], (ref["scores"] > cut)[far])
    assert np.array_equal(out["discard"][0], ref["S"]), "the case is meant to have its cut in a gap"
    C, tau = ref["C"], np.asarray(ref["tau"])[:, None]
    clear = np.all((np.abs(C - tau) > 1e-3 * tau) | (C == tau), axis=1) & (tau[:, 0] > 0)
    assert clear.sum() >= len(clear) // 4                   # (by the oracle alone: rows that the margin leaves)
    for a in np.flatnonzero(clear):
        J = ref["J"][a]
        assert np.array_equal(out["tgt"][0, a, :out["cnt"][0, a]], J)
        np.testing.assert_allclose(out["alpha"][0, a, :len(J)], ref["alpha"][a], rtol=2e-3)


def test_static_scratch_takes_what_it_took(ctx):
    """The allocation-free entry point's limit does not count the row normalisers of this form."""
    cfg = synth.ficoco_v_single(seed=9, B=16, grid=24, D=64, H=1, centres=8, dtype="bf16", n_keep=384)
    Q, K = draw_qk(10, 16, 64, 577, 32, 1.0)
    Xd, Qd, Kd = cfg["X"].to("cuda"), Q.to("cuda"), K.to("cuda")
    p = fc.make_problem(Xd, variant=fc.VARIANT_V, vis_begin=1, N=576, n_keep=384, cls_index=0, grid=(1, 24, 24), window=2,
                        Q=Qd, K=Kd, qk_begin=0)
    a, b = fc.Buffers(p, "cuda", Xd.dtype), fc.Buffers(p, "cuda", Xd.dtype)
    fc.ficoco_v_step(ctx, p, a)
    fc.ficoco_v_step_static(ctx, p, b)
    assert torch.equal(a.X_out, b.X_out) and torch.equal(a.scores, b.scores) and torch.equal(a.keep_idx, b.keep_idx)
