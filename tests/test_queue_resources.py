"""Registers of the persistent kernels for waves alone, from the built library's metadata: they leave
half of a SIMD's 512 registers to other kernels (the SIMD-exclusive form leaves none)."""
from test_kernel_resources import _find, kernels  # noqa: F401 (fixture)


def test_lone_queue_forms_leave_half_a_simd(kernels):  # noqa: F811
    lone = _find(kernels, r"k_sweeps_queue_lone")
    assert len(lone) == 6     # up to L = 8, 10, 12, plain and speculative
    for name, k in lone.items():
        assert k[".agpr_count"] == 0 and k[".vgpr_count"] <= 256, (name, k[".vgpr_count"])
        if "ELi8E" in name:
            assert k[".vgpr_count"] <= 168, (name, k[".vgpr_count"])    # three waves per SIMD, as the shared form


def test_shared_queue_form_for_small_lattices_holds_three_waves_and_no_more(kernels):  # noqa: F811
    """Where four waves fit a SIMD, a launch of three per SIMD does not spread evenly."""
    shared = _find(kernels, r"k_sweeps_queueILb[01]ELi8ELb0E")
    assert len(shared) == 2
    for name, k in shared.items():
        assert 128 < k[".vgpr_count"] <= 168 and k[".agpr_count"] == 0, (name, k[".vgpr_count"])


def test_large_tempering_kernels_spill_no_scalar_registers(kernels):  # noqa: F811
    tempering = _find(kernels, r"k_sweepsILi1[02]ELb0ELb1ELb0E")
    assert len(tempering) == 2
    for name, k in tempering.items():
        assert k.get(".sgpr_spill_count", 0) == 0, (name, k[".sgpr_spill_count"])
