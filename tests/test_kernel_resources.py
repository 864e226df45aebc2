"""The hot kernels must not use scratch memory: a register spill inside a GEMM or attention kernel costs far more than
its instruction count suggests (every reload waits for all outstanding memory operations), and nothing else in the
test suite would notice one.  Reads the per-kernel resource reports that the build keeps beside the object files
(hipcc -Rpass-analysis=kernel-resource-usage); no GPU needed."""
import json
import os

import pytest

from paper_2602_07306_amd import build as B

TILE_SOURCES = ["kernels_gemm_mfma_store.hip", "kernels_gemm_mfma_residual.hip", "kernels_gemm_mfma_swiglu.hip",
                "kernels_gemm_mfma_qkv_a.hip", "kernels_gemm_mfma_qkv_b.hip", "kernels_gemm_mfma_qkv_c.hip",
                "kernels_gemm_mfma_qkv_d.hip", "kernels_gemm_mfma_qkv_rows_a.hip",
                "kernels_gemm_mfma_qkv_rows_b.hip", "kernels_gemm_mfma_qkv_rows_c.hip"]

# kernel name fragment -> sources that instantiate it
HOT = {
    "gemm_mfma_kernel": TILE_SOURCES,
    "gemm_tile_deep_kernel": TILE_SOURCES,
    "gemm_dl_kernel": ["kernels_gemm_mfma_store.hip", "kernels_gemm_mfma_residual.hip", "kernels_gemm_mfma_swiglu.hip",
                       "kernels_gemm_mfma_qkv_a.hip", "kernels_gemm_mfma_qkv_rows_a.hip"],
    "gemm_skinny_kernel": ["kernels_gemm_skinny.hip"],
    "gemm_gemv_kernel": ["kernels_gemm_skinny.hip"],
    "attn_prefill_lds_kernel": ["kernels_attn_prefill_mfma.hip"],
    "attn_decode": ["kernels_attn_decode.hip"],
}


def load(src):
    path = B.resources_path(src)
    if not os.path.exists(path):
        pytest.skip("%s is missing: run `python -m paper_2602_07306_amd.build`" % path)
    return json.load(open(path))


@pytest.mark.parametrize("fragment", sorted(HOT))
def test_hot_kernels_use_no_scratch_memory(fragment):
    seen = 0
    for src in HOT[fragment]:
        for name, res in load(src).items():
            if fragment not in name:
                continue
            seen += 1
            assert res["ScratchSize"] == 0 and res["VGPRs Spill"] == 0, (src, name, res)
    assert seen > 0, "no kernel named *%s* in %s" % (fragment, HOT[fragment])


@pytest.mark.parametrize("fragment", ["gemm_mfma_kernel", "gemm_tile_deep_kernel", "gemm_dl_kernel"])
def test_gemm_tiles_spill_no_scalar_registers(fragment):
    """Scalar registers spill into lanes of vector registers, which the scratch test does not see.  The QKV form for rows
    of any place (the last template argument, the epilogue, is 4) is left out: it spills a few around its row table."""
    seen = 0
    for src in HOT[fragment]:
        for name, res in load(src).items():
            if fragment in name and "ELi4EEv12pt_gemm_args" not in name:
                seen += 1
                assert res["SGPRs Spill"] == 0, (src, name, res)
    assert seen > 0


def test_decode_attention_spills_no_scalar_registers():
    seen = 0
    for src in HOT["attn_decode"]:
        for name, res in load(src).items():
            if "attn_decode" in name:
                seen += 1
                assert res["SGPRs Spill"] == 0, (src, name, res)
    assert seen >= 7   # the wavefront and the workgroup form and the vector kernel at both head widths, and the combine


def test_the_square_gemm_tiles_keep_their_accumulators_in_accumulation_registers():
    """256 x 256 and 128 x 128 tiles of four wavefronts: 256 and 64 accumulators per lane.  The large ones only fit beside
    the MFMA operands, addresses and residual rows when they live in AGPRs, and the inline assembly of both ties them there."""
    big, small = {}, {}
    for src in TILE_SOURCES:
        for name, res in load(src).items():
            if "gemm_mfma_kernelILi256ELi256ELi2ELi2ELi64" in name:
                big[name] = res["AGPRs"]
            elif "gemm_mfma_kernelILi128ELi128ELi2ELi2ELi64" in name or "gemm_tile_deep_kernelILi128" in name:
                small[name] = res["AGPRs"]
    assert len(big) == 5 and all(n == 256 for n in big.values()), big      # one per epilogue
    assert len(small) == 10 and all(n >= 64 for n in small.values()), small   # two and four K steps in flight
