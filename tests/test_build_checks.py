"""The build refuses kernels on the fp64 matrix instruction whose sums the compiler puts into accumulation registers."""
import pytest

from paper_2508_02932_amd import build

LINE = "f.hip:1:1: remark: {} [-Rpass-analysis=kernel-resource-usage]\n"


def remarks(*kernels):
    return "".join(LINE.format("Function Name: " + name) + LINE.format("    VGPRs: 190") + LINE.format(f"    AGPRs: {n}") for name, n in kernels)


def test_accumulation_registers_are_found():
    ok = ("_ZN5plora10k_f32_gemmILb1EEEvi", 0), ("_ZN5plora10k_prep_f32ENS_9DescChunkE", 0), ("_ZN5plora6k_gemmEi", 128)
    assert build.kernels_with_accumulation_registers(remarks(*ok)) == []
    bad = ("_ZN5plora9k_f32_bwdILb0EEEvi", 4), ("_ZN5plora10k_prep_f32Ei", 16)
    assert build.kernels_with_accumulation_registers(remarks(*ok, *bad)) == [n for n, _ in bad]
    for nothing in ("", remarks(("_ZN5plora6k_gemmEi", 0))):
        with pytest.raises(RuntimeError):
            build.kernels_with_accumulation_registers(nothing)
