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


# images, tokens, heads, type, us of the step with the usual shape (8 lanes, rows for 512 workgroups), 32 x 8 lanes and 32 rows, 16 x 16 and 16 / 32 rows
# and 8 x 24 lanes and 32 rows
SHAPES = [
    # up to sixteen loads
    (1, 576, 8, fc.BF16, (25.9, 24.1, 25.1, 25.6, 27.2)), (3, 576, 8, fc.BF16, (28.7, 27.1, 28.1, 27.6, 28.1)), (8, 576, 12, fc.BF16, (39.7, 39.6, 40.5, 39.8, 39.7)),
    (16, 576, 16, fc.BF16, (68.9, 69.2, 70.2, 68.3, 68.9)), (8, 256, 16, fc.BF16, (26.9, 25.5, 25.4, 25.9, 28.6)),
    (8, 576, 4, fc.BF16, (31.1, 31.2, 32.5, 30.2, 31.1)), (47, 400, 4, fc.BF16, (56.2, 58.1, 59.6, 55.6, 56.2)), (48, 576, 1, fc.BF16, (71.5, 86.4, 89.8, 72.6, 71.5)),
    # more
    (1, 576, 16, fc.F32, (28.3, 26.3, 27.9, 27.8, 30.3)), (3, 400, 32, fc.F32, (33.2, 36.3, 34.7, 34.6, 37.8)), (46, 144, 40, fc.F32, (56.4, 63.1, 58.9, 63.5, 68.3)),
    (5, 428, 40, fc.F32, (52.5, 58.2, 55.3, 60.8, 53.6)), (5, 576, 40, fc.F32, (78.3, 76.5, 74.5, 73.2, 87.6)), (11, 348, 32, fc.BF16, (42.8, 45.5, 42.5, 45.6, 50.9)),
    (49, 144, 40, fc.BF16, (45.4, 48.1, 45.4, 52.6, 54.4)), (7, 465, 40, fc.BF16, (57.8, 56.9, 57.0, 56.9, 65.1)), (6, 549, 32, fc.BF16, (56.6, 55.3, 57.2, 60.5, 63.2)),
]


# Long rows, the chip nearly empty or just over one workgroup a compute unit: (the usual shape, 32 x 8), one a side.
LONG_ROWS = [
    (1, 304, 16, fc.F32, (22.8, 23.5)), (1, 304, 20, fc.F32, (23.7, 23.9)), (1, 320, 40, fc.F32, (24.8, 26.2)), (2, 288, 40, fc.F32, (25.1, 26.3)),
    (1, 448, 40, fc.F32, (28.3, 27.3)), (1, 480, 40, fc.F32, (29.6, 27.6)), (2, 376, 40, fc.F32, (28.6, 28.4)), (2, 440, 40, fc.F32, (34.2, 32.3)),
    (2, 472, 40, fc.F32, (38.9, 34.7)), (2, 488, 40, fc.F32, (40.0, 43.6)), (2, 504, 40, fc.F32, (41.1, 44.0)),
    (1, 264, 64, fc.BF16, (28.4, 27.8)), (3, 376, 64, fc.BF16, (32.9, 29.5)), (2, 488, 64, fc.BF16, (36.1, 37.7)), (2, 504, 64, fc.BF16, (38.0, 39.8)),
    (3, 658, 20, fc.BF16, (39.9, 34.5)), (9, 378, 12, fc.F32, (35.6, 34.4)), (6, 443, 40, fc.BF16, (57.7, 48.3)), (3, 660, 16, fc.F32, (44.2, 39.0)),
    (3, 510, 40, fc.F32, (59.1, 51.3)), (6, 359, 64, fc.BF16, (60.1, 49.5)), (1, 781, 48, fc.F32, (47.3, 52.3)), (5, 347, 64, fc.BF16, (38.7, 41.4)),
    (2, 1017, 40, fc.BF16, (80.4, 67.1)), (2, 918, 16, fc.F32, (55.1, 53.7)), (7, 503, 20, fc.BF16, (41.8, 41.4)),
]


@pytest.mark.parametrize("B,N,heads,dtype,us", LONG_ROWS)
def test_long_rows_take_32_by_8_only_where_it_is_no_slower(B, N, heads, dtype, us):
    r = H.reduce_plan(problem(B, N, heads, dtype))
    assert r.row_lanes in (8, 32)
    assert us[r.row_lanes == 32] <= min(1.03 * us[0], 1.05 * us[1])


# Short sequences with more than sixteen loads: (the usual shape, 16 x 16 lanes and 16 rows).
SHORT_ROWS = [
    (49, 86, 40, fc.BF16, (35.2, 29.1)), (11, 210, 32, fc.BF16, (32.4, 28.9)), (12, 219, 32, fc.F32, (36.7, 37.6)), (8, 232, 40, fc.BF16, (28.6, 27.3)),
    (5, 246, 64, fc.BF16, (31.0, 28.6)), (7, 213, 40, fc.F32, (30.2, 29.6)), (28, 129, 24, fc.F32, (30.2, 31.8)), (20, 180, 24, fc.BF16, (28.4, 30.8)),
]


@pytest.mark.parametrize("B,N,heads,dtype,us", SHORT_ROWS)
def test_short_sequences_of_many_heads_take_the_faster_shape(B, N, heads, dtype, us):
    r = H.reduce_plan(problem(B, N, heads, dtype))
    assert r.row_lanes in (8, 16)
    assert us[r.row_lanes == 16] <= 1.03 * min(us)
# Few heads, or more than 1024 columns: (the usual shape, 16 x 16 lanes and 32 rows).
TWO_ROWS = [(3, 1129, 40, fc.BF16, (124.4, 105.9)), (4, 1714, 20, fc.BF16, (149.6, 147.1)), (6, 1076, 16, fc.BF16, (93.7, 89.9)),
            (48, 576, 1, fc.BF16, (54.6, 59.2)), (47, 1145, 1, fc.BF16, (216.6, 202.0)), (13, 2082, 1, fc.F32, (184.6, 182.5)), (8, 576, 4, fc.BF16, (31.1, 30.2))]


@pytest.mark.parametrize("B,N,heads,dtype,us", TWO_ROWS)
def test_few_heads_or_long_rows_take_two_rows_a_thread_where_it_is_faster(B, N, heads, dtype, us):
    r = H.reduce_plan(problem(B, N, heads, dtype))
    assert r.row_lanes in (8, 16) and us[r.row_lanes == 16] == min(us)


@pytest.mark.parametrize("B,N,heads,dtype,us", SHAPES)
def test_shape_is_no_slower_than_the_usual(B, N, heads, dtype, us):
    r = H.reduce_plan(problem(B, N, heads, dtype))
    got = us[4 if r.rows == 32 else 0] if r.row_lanes == 8 else us[1] if r.row_lanes == 32 else us[2 if r.rows == 16 else 3]
    assert got <= 1.03 * us[0]
