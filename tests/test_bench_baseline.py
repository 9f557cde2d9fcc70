"""The benchmark's CPU baseline runs the oracle step that belongs to a workload, whatever its inputs are: maps, or the layer's
queries and keys, encoder or decoder."""
from concurrent.futures import ThreadPoolExecutor

import pytest
import torch

import bench
from paper_2411_17686_amd import ficoco as fc


def _workload(variant, qk):
    g = torch.Generator().manual_seed(1)
    B, s, N, M, H, d, D = 2, 1, 16, 3 if variant == "L" else 0, 2, 8, 12
    n = s + N + M
    st = dict(X=torch.randn(B, n, D, generator=g))
    if qk:
        st.update(Q=torch.randn(B, H, n, d, generator=g), K=torch.randn(B, H, n, d, generator=g))
    elif variant == "V":
        st.update(A=torch.softmax(torch.randn(B, H, n, n, generator=g), -1))
    else:
        st.update(A=torch.softmax(torch.randn(B, H, N, N, generator=g), -1), A_text=torch.softmax(torch.randn(B, H, M, N, generator=g), -1))
    kw = dict(vis_begin=s, N=N, n_keep=6, w_score=0.5, eps=0.9)
    kw.update(dict(cls_index=0, grid=(1, 4, 4)) if variant == "V" else dict(gamma=0.6, sem_src=fc.G_TEXT_ATTN))
    if variant == "L" and qk:
        kw["M"] = M
    return dict(sets=[st], kw=kw, B=B, N=N, d_head=d, variant=fc.VARIANT_V if variant == "V" else fc.VARIANT_L)


@pytest.mark.parametrize("qk", [False, True])
@pytest.mark.parametrize("variant", ["V", "L"])
def test_baseline_of_every_kind_of_input(variant, qk):
    with ThreadPoolExecutor(2) as pool:
        r = bench.cpu_baseline(_workload(variant, qk), pool, 2, budget=0.0)
    assert r["value"] > 0 and r["single_thread"]["value"] > 0
