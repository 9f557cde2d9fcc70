"""Orders of the workgroups of causal maps (host code; nothing is launched): every tile once, those that some query sees first; which order is taken."""
import pytest

from tests import plan_hook as H

KEYS, PER = 64, 2            # keys of a tile, tiles of a group of 128 queries


# visual tokens, text queries behind them
@pytest.mark.parametrize("N,M", [(1, 1), (63, 1), (64, 64), (127, 1), (128, 1), (129, 128), (300, 100), (576, 64), (575, 1), (640, 128), (690, 300),
                                 (704, 17), (768, 1), (1152, 300), (2881, 5), (5000, 999), (12224, 64), (12288, 1)])
def test_every_tile_once_and_live_tiles_first(N, M):
    groups, k_tiles, full = -(-(N + M) // 128), -(-N // KEYS), N // 128
    order = H.causal_tiles(groups, k_tiles, PER, full)
    assert sorted(order) == [(g, k) for g in range(groups) for k in range(k_tiles)]
    last = [min((g + 1) * 128, N + M) - 1 for g in range(groups)]          # query; those from N on see all keys
    live = [(g, k) for g in range(groups - 1, -1, -1) for k in range(k_tiles) if last[g] >= N or k * KEYS <= last[g]]
    assert order[:len(live)] == live


# images, visual tokens, text queries, us of the two kernels (32 or 40 heads of 128, of 64, of 32) with the tiles in columns and live first
MEASURED = [(8, 576, 17, (76.7, 63.4)), (8, 576, 64, (80.8, 69.8)), (8, 690, 64, (69.6, 58.8)), (8, 690, 17, (58.4, 49.2)), (8, 690, 64, (87.9, 87.5)),
            (6, 768, 200, (115.6, 140.7)), (4, 1024, 64, (80.5, 98.2)), (4, 1024, 100, (104.0, 125.4)), (3, 1152, 1, (79.0, 97.6)), (3, 1152, 100, (87.6, 106.0))]


@pytest.mark.parametrize("B,N,M,us", MEASURED)
def test_live_first_where_it_is_faster(B, N, M, us):
    k_tiles = -(-N // KEYS)
    assert us[H.causal_live_first(B * k_tiles * -(-(N + M) // 128), k_tiles)] <= 1.01 * min(us)


# images, visual tokens, text queries behind 35 others (heads of 128, 40 and 32; of 64, 32), us of the two kernels, normalisers head by head and long first
NORMALISERS = [(16, 64, 200, (58.3, 64.1)), (16, 100, 200, (63.2, 67.6)), (8, 576, 64, (86.8, 77.8)), (6, 432, 64, (48.8, 45.6)), (8, 432, 64, (44.7, 42.3)),
               (16, 576, 17, (94.6, 82.3)), (6, 690, 64, (72.8, 63.5))]


@pytest.mark.parametrize("B,N,M,us", NORMALISERS)
def test_long_groups_first_where_it_is_faster(B, N, M, us):
    def keys(query):                       # seen by it: all up to itself
        return 35 + query + 1
    first, groups = keys(191), -(-(N + M) // 192)
    if N + M - (groups - 1) * 192 <= 16:   # such a group comes behind all others
        groups -= 1
    assert us[H.causal_long_first(first, keys(min(groups * 192, N + M) - 1))] <= 1.01 * min(us)
