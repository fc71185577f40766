"""dB and dA in one launch: token walks that are split and not split, widths around the
128-column tiles, and the case in which the smaller set of partial tiles is cut to the room it has."""
import pytest

import oracle
from paper_2508_02932_amd import workloads as wl
from test_gpu_parity import run_and_compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,K,lengths,ranks,splits", [
    (136, 120, [200, 31], [16, 5], (1, 1)),                         # three stages of 64 tokens for each adapter: whole
    (128, 264, [600, 700], [16, 9], (2, 2)),
    (2048, 2560, [2048, 0, 0, 0], [16] * 4, (2, 4)),                # four splits of 64 rank rows do not fit over the skinny tiles
    (2560, 2048, [2048, 0, 0, 0], [16] * 4, (4, 2)),
])
def test_both_products_of_a_launch(D, K, lengths, ranks, splits):
    lin = wl.small(f"joint_{D}_{K}", "bf16", D, K, lengths=lengths, seg_adapter=list(range(len(lengths))), ranks=ranks,
                   scales=[2.0, 0.5, 1.0, 1.5][:len(ranks)], seed=431)
    from paper_2508_02932_amd import plora
    import gpu_harness as gh
    info, _, _ = plora.plora_debug_metadata(gh.desc_of(lin))
    assert (info.da_splits, info.db_splits) == splits
    run_and_compare(lin, impl=oracle.matmul)
