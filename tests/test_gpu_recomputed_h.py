"""A backward pass whose activation was not saved: the shrink and dH run in one launch where there is room for both sets of partial
tiles, and every result has the bits of the pass that was given the saved activation."""
import pytest

import oracle
from paper_2508_02932_amd import workloads as wl
from test_gpu_parity import run_and_compare

pytestmark = pytest.mark.gpu

MANY = [1 + 37 * i % 160 for i in range(80)]      # above 64 blocks of rows: not short
CASES = {
    "wide_in": (2504, 72, MANY, [1 + 7 * i % 40 for i in range(80)]),
    "wide_out": (72, 2504, MANY, [1 + 7 * i % 40 for i in range(80)]),
    "both_split": (1032, 2056, MANY, [16] * 80),
    "few_rows": (4104, 4096, [1] * 70 + [129], [3, 128] + [1] * 69),
}


@pytest.mark.parametrize("w_layout", [0, 1])
@pytest.mark.parametrize("case", sorted(CASES))
def test_recomputed_is_bitwise_the_saved(case, w_layout):
    import torch
    import gpu_harness as gh
    D, K, lengths, ranks = CASES[case]
    lin = wl.small(f"recomputed_{case}", "bf16", D, K, lengths=lengths, seg_adapter=list(range(len(ranks))), ranks=ranks,
                   scales=[1.0 + i % 3 for i in range(len(ranks))], seed=457)
    dp, _ = run_and_compare(lin, impl=oracle.matmul, w_layout=w_layout)
    saved = [t.clone() for t in (dp.dx, *dp.dA, *dp.dB)]
    for t in (dp.dx, *dp.dA, *dp.dB):
        t.fill_(float("nan"))
    gh.backward(dp, use_saved_h=False)
    torch.cuda.synchronize()
    gh.check_guards(dp)
    assert all(torch.equal(a, b) for a, b in zip(saved, (dp.dx, *dp.dA, *dp.dB))), case
