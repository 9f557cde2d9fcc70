"""Rows of the cosine and the Eq. 4 correlation whose targets are known from the matrix-core values alone
(the K-th largest clear of the next one) beside rows where they are not: cluster noise from far below
to far above the bound of those values, K = 1 to 6, threshold inside a gap, at a value (eps = 1), fixed K."""
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


@pytest.mark.parametrize("kw", [dict(eps=1.0), dict(eps=0.998), dict(eps=0.99), dict(eps=0.965),
                                dict(k_mode=fc.K_FIXED, fixed_k=1), dict(k_mode=fc.K_FIXED, fixed_k=3)])
@pytest.mark.parametrize("noise", [1e-4, 3e-3, 0.3])
@pytest.mark.parametrize("D,dtype", [(64, "bf16"), (520, "f32")])
def test_cosine_targets(ctx, D, dtype, noise, kw):
    cfg = synth.ficoco_v_single(seed=31, B=2, grid=17, D=D, H=2, centres=12, dtype="f32", n_keep=150)
    g = synth._gen(32)
    cfg["X"][:, 1:] = synth.clustered_tokens(g, 2, 289, D, 40, noise=noise)
    cfg["X"], cfg["A"], cfg["dtype"] = synth._cast(cfg["X"], dtype), synth._cast(cfg["A"], dtype), dtype
    kw = dict(kw, corr_src=fc.C_COSINE, k_max=64)
    out, _ = P.run_v(cfg, cfg["A"], ctx=ctx, **kw)
    for b in range(2):
        ref = P.oracle_v(cfg, cfg["A"], b, **{k: v for k, v in kw.items() if k != "k_max"})
        if max(len(j) for j in ref["J"]) > 64:            # exact duplicates: more targets than the lists hold
            assert out["overflow"][b] == 1
            continue
        P.compare_image(out, b, ref, dtype, 1, False)


@pytest.mark.parametrize("red,corr", [(fc.R_ATTN_RECV, fc.C_ATTN), (fc.R_SIM_MEAN, fc.C_COSINE)])
@pytest.mark.parametrize("M", [1, 40])
def test_decoder_targets(ctx, M, red, corr):
    cfg = synth.ficoco_l_decoder(seed=33, B=2, n_sys=3, N=200, M=M, D=264, H=2, centres=30, n_keep=70, with_vv=corr == fc.C_ATTN)
    for eps in (0.998, 0.97):
        out, _ = P.run_l(cfg, red, corr, ctx=ctx, eps=eps)
        for b in range(2):
            P.compare_image(out, b, P.oracle_l(cfg, b, red, corr, eps=eps), "bf16", cfg["vis_begin"], False)
