"""The lists of sources per target that the correlate stage of a fused step fills for the merge: targets with
fewer, exactly as many and more sources than a wavefront merges by itself (32) or a list holds (32 up to
1024 discarded tokens, 256 above), ragged widths, every way of weighting, large batches, and tokens down to
the subnormal range."""
import numpy as np
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


def sources(ref):
    n = {}
    for j in ref["J"]:
        for t in j:
            n[int(t)] = n.get(int(t), 0) + 1
    return set(n.values())


@pytest.mark.parametrize("mode", [fc.COMPRESS_SELF, fc.COMPRESS_AVERAGE])
@pytest.mark.parametrize("grid,n_keep,fixed_k,sizes", [
    (24, 50, 3, {31, 32, 33}),              # 526 discarded: around 32
    (33, 65, 2, {32, 33}),                  # 1024: the largest number of that form
    (33, 64, 2, {32, 33}),                  # 1025: the smallest of the long lists
    (48, 27, 3, {254, 258}),                # 2277: around 256
])
@pytest.mark.parametrize("D,dtype", [(72, "bf16"), (1031, "f32"), (5, "bf16")])
def test_around_the_limits(ctx, D, dtype, grid, n_keep, fixed_k, sizes, mode):
    cfg = synth.ficoco_v_single(seed=41 + grid, B=3, grid=grid, D=D, H=2, centres=9, dtype=dtype, n_keep=n_keep)
    kw = dict(corr_src=fc.C_ATTN, k_mode=fc.K_FIXED, fixed_k=fixed_k, window=2, compress_mode=mode)
    out, _ = P.run_v(cfg, cfg["A"], ctx=ctx, k_max=4, **kw)
    seen = set()
    for b in range(3):
        ref = P.oracle_v(cfg, cfg["A"], b, **kw)
        seen |= sources(ref)
        P.compare_image(out, b, ref, dtype, 1, True)
    assert any(s <= min(sizes) for s in seen) and any(s >= max(sizes) for s in seen)


def test_rows_with_many_targets(ctx):
    """Lists of up to 80 targets a row, and a target that every row names."""
    cfg = synth.ficoco_v_single(seed=47, B=2, grid=20, D=136, H=1, centres=9, dtype="f32", n_keep=160)
    cfg["A"][:, :, :, 7] = 2.0
    kw = dict(corr_src=fc.C_ATTN, k_mode=fc.K_FIXED, fixed_k=70, window=2)
    out, _ = P.run_v(cfg, cfg["A"], ctx=ctx, k_max=80, **kw)
    for b in range(2):
        ref = P.oracle_v(cfg, cfg["A"], b, **kw)
        assert max(sources(ref)) > 100
        P.compare_image(out, b, ref, "f32", 1, True)


@pytest.mark.parametrize("B,grid,n_keep", [(50, 23, 400), (100, 23, 400), (200, 23, 400), (240, 23, 400),
                                           (24, 36, 200), (60, 36, 200), (120, 36, 200)])
def test_large_batches(ctx, B, grid, n_keep):
    """Batches whose lists take many times 8 MiB: the same bytes as from the edge lists."""
    cfg = synth.ficoco_v_single(seed=53, B=2, grid=grid, D=24, H=1, centres=9, dtype="bf16", n_keep=n_keep)
    rep = (B + 1) // 2
    X, A = cfg["X"].repeat(rep, 1, 1)[:B].contiguous(), cfg["A"].repeat(rep, 1, 1, 1)[:B].contiguous()
    kw = dict(corr_src=fc.C_ATTN, k_mode=fc.K_FIXED, fixed_k=30 if grid == 23 else 8, window=2)
    one, _ = P.run_v(cfg, A, X=X, ctx=ctx, k_max=32, **kw)
    two, _ = P.run_v(cfg, A, X=X, ctx=ctx, k_max=32, staged=True, **kw)
    refs = [P.oracle_v(cfg, cfg["A"], b, **kw) for b in range(2)]
    assert max(max(sources(r)) for r in refs) <= 256
    for key in ("X_out", "pos_out", "cnt"):
        assert np.array_equal(one[key], two[key]), key
    for b in (0, 1, B - 1):
        P.compare_image(one, b, refs[b % 2], "bf16", 1, True)


@pytest.mark.parametrize("dtype,scale", [("f32", 2.0 ** -139), ("bf16", 2.0 ** -128), ("bf16", 2.0 ** 120)])
def test_extreme_tokens(ctx, dtype, scale):
    cfg = synth.ficoco_v_single(seed=59, B=1, grid=16, D=200, H=2, centres=9, dtype=dtype, n_keep=90)
    X = (cfg["X"].double() * scale).to(cfg["X"].dtype)
    kw = dict(corr_src=fc.C_ATTN, window=2)
    out, _ = P.run_v(cfg, cfg["A"], X=X, ctx=ctx, **kw)
    ref = P.oracle_v(cfg, cfg["A"], 0, X=X, **kw)
    want = P.O.widen(P.O.round_to_dtype(ref["X_out"], dtype))
    assert np.array_equal(P.O.widen(out["X_out"][0]), want)
    assert torch.isfinite(X.double()).all()


@pytest.mark.parametrize("mode", [fc.COMPRESS_SELF, fc.COMPRESS_AVERAGE])
@pytest.mark.parametrize("grid,D", [(48, 515), (33, 24), (48, 5)])
def test_one_ascending_sum_beyond_256_sources(ctx, grid, D, mode):
    """Above 1024 discarded tokens a target with more than 256 sources is one sum over ascending sources, in a
    fused step as in a staged call.  Every row names all three targets with the same weight, and every
    second source is a large number or its negative: what is left of the others depends on the order."""
    cfg = synth.ficoco_v_single(seed=61, B=1, grid=grid, D=D, H=1, centres=9, dtype="f32", n_keep=3)
    cfg["A"][:] = 0.125
    kw = dict(corr_src=fc.C_ATTN, k_mode=fc.K_FIXED, fixed_k=3, window=0, compress_mode=mode)
    S = P.oracle_v(cfg, cfg["A"], 0, **kw)["S"]
    assert len(S) > 1024
    X = cfg["X"].clone() * 1000.0
    pairs = len(S) // 4
    X[0, 1 + S[0:4 * pairs:4]] = 2.0 ** 60
    X[0, 1 + S[2:4 * pairs:4]] = -2.0 ** 60
    ref = P.oracle_v(cfg, cfg["A"], 0, X=X, **kw)
    assert sources(ref) == {len(S)}
    want = P.O.widen(P.O.round_to_dtype(ref["X_out"], "f32"))
    for staged in (True, False):
        out, _ = P.run_v(cfg, cfg["A"], X=X, ctx=ctx, k_max=4, staged=staged, **kw)
        assert np.array_equal(P.O.widen(out["X_out"][0]), want), "staged" if staged else "fused"


@pytest.mark.parametrize("staged", [False, True])
@pytest.mark.parametrize("grid,n_keep,D,dtype", [(16, 90, 72, "bf16"), (16, 90, 72, "f32"), (36, 200, 1032, "bf16"), (36, 200, 40, "f32")])
def test_infinities(ctx, grid, n_keep, D, dtype, staged):
    """Infinite features of merged tokens stay infinite (of one sign) or become NaN (of both), as the sums and the
    division of Eq. 2 give them."""
    B = 1
    cfg = synth.ficoco_v_single(seed=67, B=B, grid=grid, D=D, H=2, centres=9, dtype=dtype, n_keep=n_keep)
    X = cfg["X"].clone()
    X[0, 1::7, 0::8] = float("inf")
    X[0, 2::11, 1::8] = -float("inf")
    X[0, 3::9, 2::8] = float("inf")
    X[0, 4::9, 2::8] = -float("inf")
    kw = dict(corr_src=fc.C_ATTN, window=2)
    out, _ = P.run_v(cfg, cfg["A"], X=X, ctx=ctx, staged=staged, **kw)
    with np.errstate(invalid="ignore"):
        ref = P.oracle_v(cfg, cfg["A"], 0, X=X, **kw)
    got, want = P.O.widen(out["X_out"][0]), ref["X_out"]
    inf = np.isinf(want)
    assert inf.any() and np.isnan(want).any()
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(got[inf], want[inf])
    done = np.isfinite(want)
    assert np.array_equal(got[done], P.O.widen(P.O.round_to_dtype(want, dtype))[done])


@pytest.mark.parametrize("grid,n_keep,fixed_k", [(10, 20, 1), (10, 21, 1), (20, 1, 1), (20, 3, 2), (12, 48, 2), (12, 49, 2)])
def test_counters_packed_and_apart(ctx, grid, n_keep, fixed_k):
    """Four sources per target on average and more: the counters of the lists are 64 bytes apart, below that
    packed; here 4, just below, hundreds with one counter an image, and 4 and just below with two targets a row."""
    cfg = synth.ficoco_v_single(seed=71, B=3, grid=grid, D=40, H=2, centres=9, dtype="bf16", n_keep=n_keep)
    kw = dict(corr_src=fc.C_ATTN, k_mode=fc.K_FIXED, fixed_k=fixed_k, window=2)
    out, _ = P.run_v(cfg, cfg["A"], ctx=ctx, k_max=4, **kw)
    for b in range(3):
        P.compare_image(out, b, P.oracle_v(cfg, cfg["A"], b, **kw), "bf16", 1, True)
