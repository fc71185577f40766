"""The build refuses kernels on the fp64 matrix instruction whose sums the compiler puts into accumulation registers; and the registers that
kernels were measured with."""
import os
import re
import shutil
import subprocess

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


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not on PATH")
def test_short_products_keep_their_registers(tmp_path):
    """The preparation launch with the short products, by their blocks of 16 ranks, as it was measured (skinny_short.h)."""
    cmd = ["hipcc", *build.FLAGS, "-Rpass-analysis=" + build.REMARK, "-fno-caret-diagnostics", "--cuda-device-only", "-c",
           os.path.join(build.CSRC, "small_kernels.hip"), "-o", str(tmp_path / "small_kernels.o")]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]
    found = dict((int(n), int(v)) for n, v in re.findall(r"Function Name: \S*k_prep_shortILi(\d)E.*?\bVGPRs: (\d+)", res.stderr, re.S))
    assert sorted(found) == [1, 2, 4, 8]
    assert found[1] <= 104 and found[2] <= 102 and found[4] <= 120 and found[8] <= 168, found
