"""The filter's choice of the N^S largest scores at one and several tokens per thread (where the index sets go out
through LDS): spread scores, equal ones, few distinct ones, one far out, the ends of the range, infinities
and NaN (whose order is that of the keys: the bits of a score, the sign folded); the penalty windows of
2 x 2 with equal scores, ragged edges and empty cells; and every size of the last batch of column partials."""
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


def draw(kind, n, rng):
    x = rng.standard_normal(n)
    if kind == "equal":
        x[:] = 0.25
    elif kind == "zeros":
        x = np.where(rng.random(n) < 0.5, 0.0, -0.0)
    elif kind == "three values":
        x = rng.integers(-1, 2, n).astype(float)
    elif kind == "one far out":
        x[n // 2] = 1e9
    elif kind == "two far out":
        x[n // 3], x[n // 2] = 1e200, -1e100
    elif kind == "exponents":
        x = np.sign(x) * 10.0 ** rng.uniform(-300, 300, n)
    elif kind == "subnormal":
        x *= 1e-310
    elif kind == "largest":
        x = np.clip(x, -1, 1) * 1.7e308
    elif kind == "neighbours":
        x = 1.0 + rng.integers(0, 200, n) * 2.0 ** -52
    elif kind == "not finite":
        x[rng.random(n) < 0.1] = np.inf
        x[rng.random(n) < 0.1] = -np.inf
        x[rng.random(n) < 0.05] = np.nan
    return x


KINDS = ["spread", "equal", "zeros", "three values", "one far out", "two far out", "exponents", "subnormal", "largest",
         "neighbours", "not finite"]


def keys(x):
    u = (x + 0.0).view(np.uint64)
    return np.where(u >> np.uint64(63), ~u, u | np.uint64(1 << 63))


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("N", [1, 5, 100, 576, 1024, 1025, 2880, 4095, 4096, 12288])
def test_largest_scores(ctx, N, kind):
    rng = np.random.default_rng(N)
    X = torch.zeros(2, N + 1, 8, dtype=torch.bfloat16, device="cuda")
    vec = torch.zeros(2, 1, N, dtype=torch.bfloat16, device="cuda")
    x = np.stack([draw(kind, N, rng) for _ in range(2)])
    k = keys(x)
    for n_keep in sorted({1, N // 3, N - N // 8, N - 1, N} & set(range(1, N + 1))):
        p = fc.make_problem(X, variant=fc.VARIANT_V, vis_begin=1, N=N, n_keep=n_keep, recv_vec=vec, sem_vec=vec, window=0,
                            red_src=fc.R_VECTOR, sem_src=fc.G_VECTOR, corr_src=fc.C_COSINE, k_max=1, H=1, w_score=0.35, eps=0.998)
        buf = fc.Buffers(p, "cuda", X.dtype)
        buf.scores.copy_(torch.from_numpy(x))
        fc.ficoco_filter(ctx, p, buf)
        torch.cuda.synchronize()
        for b in range(2):
            order = np.lexsort((np.arange(N), ~k[b]))                # largest key first, then lowest index
            assert np.array_equal(buf.discard_idx[b].cpu().numpy(), np.sort(order[:N - n_keep])), n_keep
            assert np.array_equal(buf.keep_idx[b].cpu().numpy(), np.sort(order[N - n_keep:])), n_keep


@pytest.mark.parametrize("shape", [(1, 1, 9), (1, 9, 1), (2, 5, 7), (1, 24, 24), (3, 21, 19)])
@pytest.mark.parametrize("with_pos", [False, True])
def test_windows(ctx, shape, with_pos):
    f, h, w = shape
    cells, g = f * h * w, synth._gen(11)
    N = cells - (3 if with_pos else 0)
    cfg = dict(X=torch.randn(2, N, 16, generator=g).bfloat16(), B=2, H=1, D=16, n_tot=N, vis_begin=0, N=N, cls_index=-1,
               n_keep=max(1, N // 3), dtype="bf16", grid=shape, window=2, coef=2.0, lam=0.35, eps=0.998)
    for name in ("recv_vec", "sem_vec"):
        cfg[name] = (torch.randint(0, 4, (2, 1, N), generator=g) / 64).bfloat16()
    pos = torch.stack([torch.randperm(cells, generator=g)[:N].sort()[0] for _ in range(2)]).int() if with_pos else None
    kw = dict(red_src=fc.R_VECTOR, sem_src=fc.G_VECTOR, corr_src=fc.C_COSINE, pos=pos)
    out, _ = P.run_v(cfg, None, ctx=ctx, k_max=64, **kw)
    for b in range(2):
        ref = P.oracle_v(cfg, None, b, **kw)
        assert np.array_equal(out["discard"][b], ref["S"]) and np.array_equal(out["keep"][b], ref["T"])
        np.testing.assert_allclose(out["scores"][b], ref["scores"], rtol=1e-13, atol=1e-15)


@pytest.mark.parametrize("n", [9, 60, 70, 130, 200, 260, 400])
def test_column_partials(ctx, n):
    """One image: the number of row chunks grows with n, past one batch of 32."""
    cfg = synth.ficoco_v_single(seed=n, B=1, grid=1, D=16, H=1, centres=3, dtype="f32", n_keep=1)
    g = synth._gen(n)
    cfg.update(X=torch.randn(1, n + 1, 16, generator=g), A=synth.softmax_attention(g, 1, 3, n + 1, n + 1, 1.0, "f32"), N=n,
               n_tot=n + 1, H=3, n_keep=max(1, n // 2), grid=(1, 1, n))
    kw = dict(corr_src=fc.C_ATTN, window=2)
    out, _ = P.run_v(cfg, cfg["A"], ctx=ctx, **kw)
    P.compare_image(out, 0, P.oracle_v(cfg, cfg["A"], 0, **kw), "f32", 1, True)
