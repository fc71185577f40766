"""Shrink and dH of short batches: slices of 16 tokens at the edges of segments, ranks that are no multiple of 4 (A_k is read as it
lies in memory), contractions shorter than a chunk of 64, with a partial last chunk, and dealt to one and to several workgroups; both
products in the preparation launch (no saved activation), and in a launch of their own behind a long description."""
import pytest

import oracle
from paper_2508_02932_amd import plora
from paper_2508_02932_amd import workloads as wl
from test_gpu_parity import run_and_compare

pytestmark = pytest.mark.gpu

CASES = {
    "edges": (40, 72, [1, 15, 16, 17, 63, 64, 65, 129], [1, 3, 5, 16, 17, 33, 100, 128]),
    "whole_chunks": (64, 256, [16, 48, 200], [4, 16, 8]),
    "one_share": (312, 248, [130, 257, 7], [2, 64, 30]),
    "several_shares": (1000, 2504, [300, 201], [100, 7]),
    "many_shares": (4104, 520, [33], [12]),
    "rank_128": (1928, 1032, [90, 40], [128, 127]),
    "rank_128_long_rows": (2056, 1032, [90, 40], [128, 127]),     # a third chunk for a wave: the shrink is not short
}
SHARES = {"edges": (1, 1), "whole_chunks": (1, 1), "one_share": (1, 1), "several_shares": (4, 5), "many_shares": (8, 2), "rank_128": (4, 4),
          "rank_128_long_rows": (0, 4)}


def gh():
    import gpu_harness
    return gpu_harness


@pytest.mark.parametrize("w_layout", [0, 1])
@pytest.mark.parametrize("save_h", [True, False])
@pytest.mark.parametrize("case", sorted(CASES))
def test_short(case, save_h, w_layout):
    D, K, lengths, ranks = CASES[case]
    lin = wl.small(f"short_{case}", "bf16", D, K, lengths=lengths, seg_adapter=list(range(len(ranks))), ranks=ranks,
                   scales=[2.0, 0.5, 1.25, 1.0, 3.0, 4.0, 0.25, 1.5][:len(ranks)], seed=443)
    assert tuple(plora.plora_debug_metadata(gh().desc_of(lin, w_layout))[0].short_shares) == SHARES[case]
    run_and_compare(lin, impl=oracle.matmul, save_h=save_h, w_layout=w_layout)


@pytest.mark.parametrize("save_h", [True, False])
def test_short_behind_a_long_description(save_h):
    """Half of the adapters have no tokens: at most 64 token blocks, but more words than a kernel argument carries.  The products
    take a launch of their own, shrink on the packed A_k^T, dH behind it on the same partial sums and flags."""
    n = 90
    lin = wl.small("short_long_description", "bf16", 1000, 2504, lengths=[1 + i % 20 if i % 2 else 0 for i in range(n)],
                   seg_adapter=list(range(n)), ranks=[1 + 5 * i % 48 for i in range(n)], scales=[1.0 + i % 3 for i in range(n)], seed=449)
    info = plora.plora_debug_metadata(gh().desc_of(lin))[0]
    assert info.n_blocks <= 64 and info.desc_words > 896 and min(info.short_shares) > 1
    run_and_compare(lin, impl=oracle.matmul, save_h=save_h)


def test_not_short_behind_a_long_description():
    n = 90
    lin = wl.small("long_description", "bf16", 328, 264, lengths=[1 + i % 20 for i in range(n)], seg_adapter=list(range(n)),
                   ranks=[1 + 5 * i % 64 for i in range(n)], scales=[1.0 + i % 3 for i in range(n)], seed=449)
    info = plora.plora_debug_metadata(gh().desc_of(lin))[0]
    assert info.n_blocks > 64 and info.desc_words > 896 and list(info.short_shares) == [0, 0]
    run_and_compare(lin, impl=oracle.matmul, save_h=False)


def test_neither_product_is_short():
    """More than 64 token blocks: the kernel for long batches, with segments and ranks at the same edges."""
    lin = wl.small("not_short", "bf16", 1032, 1544, lengths=[1, 15, 16, 17, 63, 64, 65, 129] + [1 + i % 9 for i in range(64)],
                   seg_adapter=[i % 8 for i in range(72)], ranks=[1, 3, 5, 16, 17, 33, 100, 128],
                   scales=[2.0, 0.5, 1.25, 1.0, 3.0, 4.0, 0.25, 1.5], seed=449)
    info = plora.plora_debug_metadata(gh().desc_of(lin))[0]
    assert list(info.short_shares) == [0, 0] and min(info.shrink_splits, info.dh_splits) > 1
    for save_h in (True, False):
        run_and_compare(lin, impl=oracle.matmul, save_h=save_h)
