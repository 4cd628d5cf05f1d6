"""Registers of the kernels as built: what a launch relies on to have several workgroups on a compute unit beside each other."""
import re

from tests.test_kernel_args import kernels


def waves(kernel):
    """wavefronts a SIMD of 512 registers a lane holds, given out in eights"""
    return min(8, 512 // ((kernel[".vgpr_count"] + 7) // 8 * 8))


GEMM = re.compile(r"11gemm_kernelILi(.)ELi.ELi.ELi.ELi(\d+)ELi(.)ELb(.)ELb(.)ELb(.)E.*Gemm(Args|Pair)")


# the grouped GEMM on 64 columns and 32-deep slabs: six without a residual, linear layers, strided ones and pairs, bf16 and fp32 results
def test_short_slabs_of_the_grouped_gemm():
    found = {m.groups(): k for m, k in ((GEMM.search(n), k) for n, k in kernels().items()) if m}
    short = {g[3:]: k for g, k in found.items() if g[:3] == ("4", "32", "1") and g[4] == "0"}
    assert set(short) == {("0", "0", "0", "Args"), ("0", "0", "1", "Args"), ("1", "0", "0", "Args"), ("1", "0", "0", "Pair")}
    for name, k in short.items():
        assert waves(k) >= 6, name
    for name, k in found.items():
        assert k[".private_segment_fixed_size"] == 0, name


# transformer blocks with two workgroups of four wavefronts a compute unit: two wavefronts a SIMD, and nothing in scratch up to 384 channels (what waits
# there is waited for like the operands asked for before it), above them, with four column blocks a wavefront, two registers a lane at most
def test_transformer_blocks_of_two_workgroups():
    found = {n: k for n, k in kernels().items() if "vit_duo_kernel" in n}
    assert len(found) == 2
    for name, k in found.items():
        assert waves(k) >= 2, name
        assert k[".private_segment_fixed_size"] <= (8 if "Li416E" in name else 0), name


# 3x3 layers on tiled filters: two wavefronts a SIMD, nothing in scratch
def test_tiled_3x3_layers():
    found = {n: k for n, k in kernels().items() if "conv3_tiled_kernel" in n}
    assert len(found) == 3
    for name, k in found.items():
        assert waves(k) >= 2 and k[".private_segment_fixed_size"] == 0, name
