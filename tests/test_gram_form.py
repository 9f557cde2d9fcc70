"""Which tiles the block of approximate cosines is cut into (host code; nothing is launched)."""
from paper_2411_17686_amd import ficoco as fc
from tests import plan_hook as H


def plan(B, n_disc, n_keep, D):
    p = fc.Problem()
    N = n_disc + n_keep
    p.variant, p.dtype = fc.VARIANT_V, fc.BF16
    p.B, p.H, p.D, p.n_tot, p.N, p.n_keep, p.cls_index = B, 1, D, N, N, n_keep, -1
    p.X, p.x_stride_b, p.x_stride_n, p.recv_vec, p.sem_vec = 4096, N * D, D, 4096, 4096
    p.red_src, p.sem_src, p.corr_src = fc.R_VECTOR, fc.G_VECTOR, fc.C_COSINE
    p.eps, p.gamma, p.w_score, p.k_max = 0.998, 0.6, 0.35, 8
    g = H.gram_plan(p)
    assert g.use_gram
    return g


def test_images_of_four_gib_keep_large_tiles():
    """The 192-row tiles address an image's rows with 32 bits: the taller ones, with 64, take over at 4 GiB."""
    below, beyond = plan(1, 11136, 1152, 174760), plan(1, 11136, 1152, 174768)
    assert below.splits == 1 and below.form != H.SQUARE
    assert beyond.splits == 1 and beyond.form == H.TALL
