"""Registers of the kernels as built: what a launch relies on to have several workgroups on a compute unit beside each other."""
import re

from tests.test_kernel_args import kernels


def waves(kernel):
    """wavefronts a SIMD of 512 registers a lane holds, given out in eights"""
    return min(8, 512 // ((kernel[".vgpr_count"] + 7) // 8 * 8))


# the grouped GEMM on 64 columns and 32-deep slabs: six without a residual, linear layers, strided ones and pairs alike
def test_short_slabs_of_the_grouped_gemm():
    form = re.compile(r"11gemm_kernelILi4ELi1ELi1ELi2ELi32ELi1ELb(.)ELb0E.*Gemm(Args|Pair)")
    found = {m.groups(): k for m, k in ((form.search(n), k) for n, k in kernels().items()) if m}
    assert set(found) == {("0", "Args"), ("1", "Args"), ("1", "Pair")}
    for name, k in found.items():
        assert waves(k) >= 6 and k[".private_segment_fixed_size"] == 0, name
