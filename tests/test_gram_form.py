"""Which tiles the block of approximate cosines is cut into (host code; nothing is launched)."""
import pytest

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


# images, discarded, kept, features, us with tiles of 128 x 128, 192 x 192 and (one K range) 256 x 192, measured one after the other
MEASURED = [
    # padding, short K, many images
    (260, 98, 98, 128, (8.7, 19.0, 16.0)), (260, 480, 96, 128, (20.0, 39.5, 28.4)), (180, 200, 200, 128, (12.7, 24.7, 18.5)),
    (64, 200, 200, 256, (10.2, 11.6, 12.3)), (128, 432, 144, 256, (21.2, 24.4, 15.8)), (40, 700, 200, 128, (10.5, 18.9, 11.1)),
    # one round of the larger tiles, or two with a nearly empty second
    (1, 8064, 1152, 1024, (38.7, 27.4, 33.3)), (1, 8064, 1152, 4096, (122.0, 73.5, 100.3)), (1, 10368, 1152, 1024, (39.7, 43.6, 35.2)),
    (36, 768, 384, 1024, (38.1, 43.0, 33.8)), (44, 768, 384, 1024, (56.5, 44.5, 59.1)), (2, 8064, 1152, 1024, (63.8, 50.6, 63.5)),
    # long K
    (36, 768, 384, 4096, (154.6, 159.5, 122.7)), (90, 432, 144, 4096, (147.0, 150.0, 120.8)),
    # several K ranges
    (16, 768, 384, 1024, (23.5, 19.5)), (16, 768, 384, 4096, (64.8, 43.2)), (64, 384, 192, 1024, (24.0, 22.0)), (8, 432, 144, 4096, (17.5, 18.0)),
]


@pytest.mark.parametrize("B,n_disc,n_keep,D,us", MEASURED)
def test_form_is_among_the_fastest(B, n_disc, n_keep, D, us):
    """Within 7 % of the fastest: the usual form is only left for one clearly faster by estimate."""
    g = plan(B, n_disc, n_keep, D)
    assert (g.splits > 1) == (len(us) == 2)
    assert us[g.form] <= 1.07 * min(us)


def test_images_of_four_gib_keep_large_tiles():
    """Rows beyond 4 GiB of an image are addressed like any others."""
    below, beyond = plan(1, 11136, 1152, 174752), plan(1, 11136, 1152, 174784)
    assert below.splits == 1 and beyond.splits == 1
    assert below.form == beyond.form != H.SQUARE
