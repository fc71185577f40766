"""dH of a batch that is not short in the launch of the preparation: more segments than a wave has lanes, repeated and empty segments,
rows of the base model alone, ranks and widths that fill no tile, rank 128, against the fp64 oracle; a call with far more packing than dH
keeps two launches.  Tolerance as in test_gpu_parity.py."""
import pytest

import oracle
from paper_2508_02932_amd import plora
from paper_2508_02932_amd import workloads as wl
from test_gpu_parity import run_and_compare

pytestmark = pytest.mark.gpu

CASES = {
    # d_in, d_out, lengths, owners, ranks, launches of the preparation alone
    "many_segments": (136, 200, [1 + i % 130 for i in range(100)], [i % 5 if i % 9 else -1 for i in range(100)], [3, 8, 17, 64, 100], 0),
    "edges": (520, 1032, [127, 128, 129, 0, 8000, 300, 1], [0, 1, 2, 0, 1, -1, 2], [1, 128, 33], 0),
    "whole_lines": (1024, 512, [5000, 4000], [1, 0], [16, 64], 0),
    "much_packing": (8192, 264, [90] + [0] * 39, list(range(40)), [128] + [64] * 39, 1),
}


@pytest.mark.parametrize("w_layout", [0, 1])
@pytest.mark.parametrize("case", sorted(CASES))
def test_dh(case, w_layout):
    import torch
    import gpu_harness as gh
    D, K, lengths, owner, ranks, launches = CASES[case]
    lin = wl.small(f"prep_dh_{case}", "bf16", D, K, lengths=lengths, seg_adapter=owner, ranks=ranks, scales=[2.0, 0.5, 1.25, 1.0, 3.0][:len(ranks)] + [1.0] * (len(ranks) - 5),
                   seed=487)
    info = plora.plora_debug_metadata(gh.desc_of(lin, w_layout))[0]
    assert info.short_shares[1] == 0 and info.desc_words <= 896
    dp, _ = run_and_compare(lin, impl=oracle.matmul, w_layout=w_layout)
    plora.plora_set_kernel_timing(True)
    try:
        gh.backward(dp)
        torch.cuda.synchronize()
        assert (plora.plora_kernel_time(6)[1], plora.plora_kernel_time(3)[1]) == (launches, 1)
    finally:
        plora.plora_set_kernel_timing(False)
