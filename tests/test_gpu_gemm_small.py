"""The base GEMM in small tiles with the contraction split over workgroups: sizes at the edges of its tiles (64 or 128 rows,
128 columns, 64 contraction elements), splits with a partial last step, row tiles with more segments than one wave's window
of 64 records, both weight orders, and the accumulating epilogue of a grouped call, against the fp64 oracle.  Tolerance:
the bf16 one of test_gpu_parity.py (2e-2 scaled; output rounding 2^-9 and the bf16 rounding of h and g)."""
import numpy as np
import pytest

from paper_2508_02932_amd import workloads as wl
from test_gpu_parity import run_and_compare

pytestmark = pytest.mark.gpu


def tokens_of(n, parts):
    return [n // parts + (i < n % parts) for i in range(parts)]


CASES = {
    # T, D, K, segments
    "one_token": (1, 512, 1024, 1),
    "tile_minus_1": (63, 1032, 136, 3),
    "tile_plus_1": (65, 2056, 120, 4),
    "two_tiles_split": (129, 4104, 264, 5),
    "wide_128_rows": (513, 1096, 14344, 3),          # 128-row tiles, partial last column tile
    "deep_128_rows": (514, 14344, 1096, 3),          # the same in the other direction, contraction split
    "many_segments": (200, 776, 520, 150),           # more than 64 segments in a row tile
}


@pytest.mark.parametrize("w_layout", [0, 1])
@pytest.mark.parametrize("case", sorted(CASES))
def test_small_tiles(case, w_layout):
    import oracle
    T, D, K, parts = CASES[case]
    n_ad = min(parts, 7)
    owner = [(-1 if i % 11 == 10 else i % n_ad) for i in range(parts)]
    lin = wl.small(f"gemm_small_{case}", "bf16", D, K, lengths=tokens_of(T, parts), seg_adapter=owner,
                   ranks=[8, 33, 64, 1, 128, 17, 72][:n_ad], scales=[2.0, 0.5, 1.0, 4.0, 0.25, 1.5, 2.0][:n_ad], seed=211)
    run_and_compare(lin, impl=oracle.matmul, w_layout=w_layout)


def test_more_than_64_segments_in_the_call_and_in_a_later_row_tile():
    import oracle
    lengths = [1] * 100 + [0] * 20 + [2] * 140 + [70]
    lin = wl.small("gemm_small_windows", "bf16", 520, 392, lengths=lengths, seg_adapter=[i % 5 for i in range(len(lengths))],
                   ranks=[8, 72, 3, 128, 40], scales=[2.0] * 5, seed=223)
    run_and_compare(lin, impl=oracle.matmul)


@pytest.mark.parametrize("w_layout", [0, 1])
@pytest.mark.parametrize("D,K,tail", [(264, 648, 77), (512, 512, 12501)])
def test_256_row_tiles_with_several_segments_and_ragged_edges(D, K, tail, w_layout):
    """Enough row tiles for the 256 x 256 kernel: tiles with one, two and more than two segments, partial last tiles and step.
    35336 tokens: whole rounds in 256-row tiles and the rest of the row tiles (in the order that kernel walks them) in small
    ones; 32760 tokens, 512 -> 512: one full round."""
    import oracle
    lengths = [300, 7, 90, 0, 61, 4000, 1, 2, 30, 9000, 255, 513, 21000 if tail == 77 else 6000, tail]
    lin = wl.small(f"gemm_256_ragged_{D}", "bf16", D, K, lengths=lengths, seg_adapter=[i % 4 if i % 6 else -1 for i in range(len(lengths))],
                   ranks=[8, 72, 3, 128], scales=[2.0, 1.0, 0.5, 0.25], seed=229)
    run_and_compare(lin, impl=oracle.matmul, w_layout=w_layout)


def test_workspace_of_a_call_that_fits_the_scratch_array_does_not_outgrow_it():
    from paper_2508_02932_amd import plora
    import gpu_harness as gh
    lin = wl.small("gemm_small_scratch", "bf16", 8192, 8192, lengths=[512], seg_adapter=[0], ranks=[128], scales=[1.0], seed=227)
    assert plora.plora_workspace_bytes(gh.desc_of(lin)) <= plora.NOALLOC_SCRATCH_BYTES
