"""Kernel-class names of the layer and conv instantiations, from the symbols a trace holds."""
import pytest

from paper_2208_05740_amd.profiling import class_of


@pytest.mark.parametrize("symbol,name", [
    ("void gcp::layer_kernel<float, 1, 1, 2, 2, 0, false, gcp::AdjEpi<float, false> >", "adj.fp32.t32x32"),
    ("void gcp::layer_kernel<float, 1, 1, 1, 4, 3, true, gcp::AdjEpi<float, false> >", "adj.fp32.sign.t16x64d"),
    ("_ZN3gcp12layer_kernelIDF16bLi1ELi2ELi2ELi2ELi0ELb0ENS_8BoundEpiIDF16bLb0EEEEEvNS_8GemmArgsET6_", "bound.bf16.t32x64"),
    ("_ZN3gcp12layer_kernelIDF16bLi1ELi1ELi1ELi2ELi4ELb0ENS_7ConcEpiEEEvNS_8GemmArgsET6_", "conc.bf16.t16x32d"),
    ("void gcp::conv_slab_kernel<float, 8, 1, 4, true, false, gcp::BoundEpi<float, false> >", "convT_bound.fp32.w8x1"),
    ("_ZN3gcp16conv_slab_kernelIDF16bLi4ELi2ELi1ELb0ELb1ENS_6AdjEpiIDF16bLb0EEEEEvNS_8ConvArgsENS_8ConvPlanET5_i",
     "conv_adj.bf16.sign.w4x2"),
])
def test_class_names(symbol, name):
    assert class_of(symbol) == name
