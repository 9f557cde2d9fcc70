"""Registers of the built kernels, from the notes of the code objects in the library: what a kernel was written to hold in
registers does not go over scratch memory or lanes of vector registers."""
import os
import re
import subprocess

import pytest

from paper_2411_17686_amd import ficoco as fc

LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{name: {vgpr_count, sgpr_spill_count, vgpr_spill_count, private_segment_fixed_size}} of every kernel."""
    d = tmp_path_factory.mktemp("objects")
    lib = d / "libficoco.so"
    lib.symlink_to(fc.LIB_PATH)
    subprocess.run([os.path.join(LLVM, "llvm-objdump"), "--offloading", str(lib)], cwd=d, check=True, stdout=subprocess.DEVNULL)
    found = {}
    for f in sorted(os.listdir(d)):
        if "gfx950" not in f:
            continue
        notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", str(d / f)], check=True, capture_output=True, text=True).stdout
        for k in re.split(r"\n\s+- \.agpr_count:", notes)[1:]:
            name = re.search(r"\.name:\s+(\S+)", k).group(1)
            found[name] = {n: int(re.search(r"\.%s:\s+(\d+)" % n, k).group(1))
                           for n in ("vgpr_count", "sgpr_spill_count", "vgpr_spill_count", "private_segment_fixed_size")}
    assert len(found) > 60
    return found


def _all(kernels, part):
    got = {n: r for n, r in kernels.items() if part in n}
    assert got, part
    return got


def test_candidate_rows_keep_their_scalars(kernels):
    for n, r in _all(kernels, "corr_cand_rows_kernel").items():
        assert r["sgpr_spill_count"] == r["vgpr_spill_count"] == r["private_segment_fixed_size"] == 0, (n, r)


def test_head_mean_of_queries_and_keys_uses_no_scratch(kernels):
    for n, r in _all(kernels, "qk_mean_kernel").items():
        assert r["vgpr_spill_count"] == r["private_segment_fixed_size"] == 0, (n, r)


@pytest.mark.parametrize("part", ["qk_mean_deep_kernel", "qk_norm_kernel", "unit_rows_kernel", "unit_terms_kernel", "unit_mean_kernel",
                                  "attn_reduce_kernel", "attn_text_reduce_kernel", "gram_tile_kernel"])
def test_other_kernels_use_no_scratch(kernels, part):
    for n, r in _all(kernels, part).items():
        assert r["vgpr_spill_count"] == r["private_segment_fixed_size"] == 0, (n, r)


def test_reduction_of_bfloat16_maps_keeps_four_wavefronts_a_simd(kernels):
    """The instances with 16-byte rows of bfloat16 (one more register than 128 is a quarter of the wavefronts)."""
    for part in ("18attn_reduce_kernelIt", "23attn_text_reduce_kernelIt"):
        for n, r in _all(kernels, part).items():
            assert r["vgpr_count"] <= 128, (n, r)


def test_head_mean_of_one_block_has_nothing_else(kernels):
    """Causal heads of 128, not split: launched with one block of queries only, without the registers of whole tiles."""
    (n, r), = _all(kernels, "qk_mean_kernelILi4ELb1ELb0E").items()
    assert r["vgpr_count"] <= 128, (n, r)
