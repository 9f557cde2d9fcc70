"""How the reduction of maps is cut and who adds its column partials (host code; nothing is launched)."""
import pytest

from paper_2411_17686_amd import ficoco as fc
from tests import plan_hook as H


def problem(B, N, heads, dtype=fc.BF16, n_keep=None, maps=True, Df=0):
    """One [CLS] row in front of N visual tokens; maps or (64 features) queries and keys; Df: the mean feature row as the score's other term."""
    p = fc.Problem()
    n = N + 1
    p.variant, p.dtype = fc.VARIANT_V, dtype
    p.B, p.H, p.D, p.n_tot, p.vis_begin, p.N, p.n_keep, p.cls_index = B, heads, 64, n, 1, N, n_keep or max(1, N // 2), 0
    p.X, p.x_stride_b, p.x_stride_n = 4096, n * 64, 64
    if maps:
        p.A, p.a_stride_b, p.a_stride_h, p.a_stride_q, p.a_nq, p.a_nk = 4096, heads * n * n, n * n, n, n, n
    else:
        p.Q = p.K = 4096
        p.qk_stride_b, p.qk_stride_h, p.qk_stride_n, p.qk_n, p.d_head, p.qk_dtype, p.qk_scale = heads * n * 64, n * 64, 64, n, 64, fc.BF16, 0.125
    if Df:
        p.F, p.f_stride_b, p.f_stride_n, p.Df = 4096, N * Df, Df, Df
    p.red_src, p.sem_src, p.corr_src = fc.R_ATTN_RECV, fc.G_EQ_TOKEN if Df else fc.G_CLS_ATTN, fc.C_ATTN
    p.eps, p.gamma, p.w_score, p.k_max = 0.998, 0.6, 0.35, 8
    return p


# images, tokens, heads, from maps, us behind the reduction with the partials added by the filter and by a launch of their own
PARTIALS = [(1, 640, 4, True, (16.3, 16.4)), (4, 1025, 4, True, (30.9, 29.9)), (1, 1296, 4, True, (31.4, 28.4)), (4, 1296, 4, True, (35.7, 32.9)),
            (1, 1728, 4, True, (36.5, 30.2)), (4, 1728, 4, True, (44.7, 38.4)), (1, 2000, 4, True, (41.5, 30.6)),
            (1, 1440, 4, False, (27.9, 27.8)), (1, 1728, 4, False, (31.6, 28.8)), (1, 2304, 4, False, (47.6, 40.5)), (3, 2500, 4, False, (65.3, 57.0))]


@pytest.mark.parametrize("B,N,heads,maps,us", PARTIALS)
def test_many_partials_are_added_by_a_launch_of_their_own(B, N, heads, maps, us):
    r = H.reduce_plan(problem(B, N, heads, maps=maps))
    assert us[r.combined] <= 1.02 * min(us)


# images, tokens, edges a token at most: just within the limit with chunks of 24 rows, beyond it with 16
LARGEST = [(64, 128, 580), (16, 256, 1167), (85, 96, 586)]


@pytest.mark.parametrize("B,N,k_max", LARGEST)
def test_static_scratch_holds_the_partials_of_small_maps(B, N, k_max):
    """A step's workspace, without its lists, is within the limit of the allocation-free entry point."""
    p = problem(B, N, 8)
    p.k_max = k_max
    r = H.reduce_plan(p, 48 << 20)
    assert r.total - r.beyond <= fc.STATIC_SCRATCH_BYTES
