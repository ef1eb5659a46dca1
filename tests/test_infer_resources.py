"""Registers of the BF16 inference of up to 8192 rows, from the built library's metadata: its eight
waves, two per SIMD, fit beside waves that hold half of a SIMD's 512 registers."""
from test_kernel_resources import _find, kernels  # noqa: F401 (fixture)


def test_inference_of_one_tile_per_workgroup_leaves_half_a_simd(kernels):  # noqa: F811
    (name, k), = _find(kernels, r"k_infer_bf16ILb0E").items()
    assert k[".vgpr_count"] <= 128 and k[".agpr_count"] == 0, (name, k[".vgpr_count"])
    assert k.get(".vgpr_spill_count", 0) == 0 and k.get(".private_segment_fixed_size", 0) == 0
