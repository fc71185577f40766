"""The fp32 path at the edges of its tiles (16 and 32 rows, 32 columns, 16 and 32 contraction elements, 16 ranks): sizes one below
and above them, rows that are not 16-byte aligned, ranks from 1 to 128, segments shorter than a tile, both weight orders,
against the fp64 oracle.  Tolerance 1e-5 as for every fp32 call (sums are in fp64, results rounded to fp32: 6e-8)."""
import pytest

from paper_2508_02932_amd import workloads as wl
from test_gpu_parity import run_and_compare

pytestmark = pytest.mark.gpu

CASES = {
    "below": (31, 31, 63, [31], [0], [31]),
    "above": (33, 33, 65, [16, 17], [1, 0], [33, 1]),
    "one": (1, 1, 1, [1], [0], [1]),
    "deep": (40, 1027, 18, [7, 0, 33], [0, 1, 1], [128, 100]),
    "wide": (300, 18, 1030, [1, 2, 3, 130, 164], [0, 1, -1, 2, 0], [17, 64, 5]),
    "row_tiles": (545, 100, 97, [255, 2, 31, 257], [0, 1, 2, 0], [16, 32, 48]),
}


@pytest.mark.parametrize("w_layout", [0, 1])
@pytest.mark.parametrize("save_h", [True, False])
@pytest.mark.parametrize("case", sorted(CASES))
def test_f32_tile_edges(case, save_h, w_layout):
    T, D, K, lengths, owner, ranks = CASES[case]
    assert sum(lengths) == T
    lin = wl.small(f"f32_{case}", "f32", D, K, lengths=lengths, seg_adapter=owner, ranks=ranks, scales=[1.5] * len(ranks), seed=307)
    run_and_compare(lin, save_h=save_h, w_layout=w_layout)


SIDES = {   # 16 x 16 output tiles up to 1024 of them, 32 x 32 above; contractions around one and two chunks of 16
    "small_tiles": (512, 512, 512, [200, 312], [0, 1], [16, 9]),
    "large_tiles": (515, 31, 530, [500, 15], [0, 1], [17, 3]),                # the last segment ends in a row tile of three rows
    "large_forward": (700, 16, 400, [333, 0, 367], [1, 0, -1], [5, 20]),
    "large_backward": (1040, 300, 15, [7, 1000, 33], [0, 1, 2], [48, 1, 16]),
    "one_chunk": (530, 17, 500, [17, 513], [0, 1], [15, 16]),
}


@pytest.mark.parametrize("w_layout", [0, 1])
@pytest.mark.parametrize("case", sorted(SIDES))
def test_f32_tile_sides(case, w_layout):
    import oracle
    T, D, K, lengths, owner, ranks = SIDES[case]
    lin = wl.small(f"f32_{case}", "f32", D, K, lengths=lengths, seg_adapter=owner, ranks=ranks, scales=[1.5] * len(ranks), seed=313)
    assert lin.layout.T == T
    run_and_compare(lin, impl=oracle.matmul, w_layout=w_layout)


def test_f32_infinity_stays_in_its_own_rows():
    """An infinity in one adapter's B reaches the rows of that adapter's segments and no other row of the same tile."""
    import numpy as np
    import torch
    import gpu_harness as gh
    lin = wl.small("f32_inf", "f32", 40, 48, lengths=[10, 9, 13], seg_adapter=[0, 1, 0], ranks=[4, 6], scales=[1.0, 1.0], seed=311)
    t = lin.tensors()
    clean, dirty = gh.upload(lin, t), gh.upload(lin, t)
    dirty.B[1][2, 5] = float("inf")
    for dp in (clean, dirty):
        gh.forward(dp)
    torch.cuda.synchronize()
    a, b = gh.to_np(clean.y), gh.to_np(dirty.y)
    other = np.r_[0:10, 19:32]
    assert np.array_equal(a[other], b[other])
    assert not np.isfinite(b[10:19, 5]).any()
