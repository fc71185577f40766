"""The base GEMM in small tiles with the contraction split over workgroups: sizes at the edges of its tiles (64 or 128 rows,
128 columns, 64 contraction elements), splits with a partial last step, row tiles with more segments than one wave's window
of 64 records, both weight orders, and the accumulating epilogue of a grouped call, against the fp64 oracle.  Tolerance:
the bf16 one of test_gpu_parity.py (2e-2 scaled; output rounding 2^-9 and the bf16 rounding of h and g).  What a product runs
on is a function of its sizes (the plan); the cases say which plan they are about and check it: (rows of the small tiles, 0:
256 x 256 tiles alone; splits of the contraction; row tiles left to the 256 x 256 kernel)."""
import numpy as np
import pytest

from paper_2508_02932_amd import workloads as wl
from test_gpu_parity import run_and_compare

pytestmark = pytest.mark.gpu


def tokens_of(n, parts):
    return [n // parts + (i < n % parts) for i in range(parts)]


def plan_of(lin, w_layout=0):
    import gpu_harness as gh
    from paper_2508_02932_amd import plora
    info, _, _ = plora.plora_debug_metadata(gh.desc_of(lin, w_layout))
    return [(info.gemm_rows[i], info.gemm_splits[i], info.gemm_big_tiles[i]) for i in range(2)]


def ragged(name, T, D, K, parts, seed, ranks=(8, 33, 64, 1, 128, 17, 72), scales=(2.0, 0.5, 1.0, 4.0, 0.25, 1.5, 2.0)):
    """T tokens in `parts` segments, every eleventh of the base model alone, the others dealt to up to seven adapters."""
    n_ad = min(parts, 7)
    owner = [(-1 if i % 11 == 10 else i % n_ad) for i in range(parts)]
    return wl.small(name, "bf16", D, K, lengths=tokens_of(T, parts), seg_adapter=owner, ranks=list(ranks[:n_ad]), scales=list(scales[:n_ad]),
                    seed=seed)


CASES = {
    # T, D, K, segments
    "one_token": (1, 512, 1024, 1),
    "tile_minus_1": (63, 1032, 136, 3),
    "tile_plus_1": (65, 2056, 120, 4),
    "two_tiles_split": (129, 4104, 264, 5),
    "wide": (513, 1096, 14344, 3),                   # partial last column tile
    "wide_contraction": (514, 14344, 1096, 3),       # the same in the other direction
    "many_segments": (200, 776, 520, 150),           # more than 64 segments in a row tile
}


@pytest.mark.parametrize("w_layout", [0, 1])
@pytest.mark.parametrize("case", sorted(CASES))
def test_small_tiles(case, w_layout):
    import oracle
    lin = ragged(f"gemm_small_{case}", *CASES[case], 211)
    assert all(rows == 64 and big == 0 for rows, _, big in plan_of(lin, w_layout))
    run_and_compare(lin, impl=oracle.matmul, w_layout=w_layout)


PLANS = {
    # T, D, K, segments, plan of the forward product, plan of dX.  128-row tiles up to 512 tokens: a third slot of the W ring
    "ring_of_three": (511, 1096, 14344, 3, (128, 1, 0), (64, 7, 0)),
    "ring_of_three_split": (200, 4104, 8200, 5, (128, 3, 0), (128, 5, 0)),
    "ring_of_three_many_segments": (200, 8200, 4104, 190, (128, 5, 0), (128, 3, 0)),     # the window of 64 records is moved back and forth
    "128_rows": (1023, 4104, 4104, 6, (128, 1, 0), (128, 1, 0)),
    "128_rows_split": (700, 4104, 8200, 4, (128, 1, 0), (128, 2, 0)),
    "128_rows_split_many_segments": (700, 8200, 4104, 300, (128, 2, 0), (128, 1, 0)),
    "rest_in_64_rows": (2047, 520, 8200, 9, (64, 1, 7), (64, 3, 0)),
    "rest_in_64_rows_many_segments": (2047, 8200, 520, 900, (64, 3, 0), (64, 1, 7)),
    "rest_in_128_rows": (9000, 520, 2056, 9, (128, 1, 28), (128, 1, 0)),
    "rest_in_128_rows_dx": (9000, 2056, 520, 100, (128, 1, 0), (128, 1, 28)),
}


@pytest.mark.parametrize("w_layout", [0, 1])
@pytest.mark.parametrize("case", sorted(PLANS))
def test_planned_tiles(case, w_layout):
    import oracle
    T, D, K, parts, fwd, dx = PLANS[case]
    lin = ragged(f"gemm_plan_{case}", T, D, K, parts, 233)
    assert plan_of(lin, w_layout) == [fwd, dx]
    run_and_compare(lin, impl=oracle.matmul, w_layout=w_layout)


@pytest.mark.parametrize("w_layouts", [(0, 0), (1, 1)])
@pytest.mark.parametrize("case", ["ring_of_three_split", "ring_of_three_many_segments", "128_rows", "128_rows_split", "rest_in_64_rows_many_segments",
                                  "rest_in_128_rows_dx"])
def test_planned_tiles_accumulating(case, w_layouts):
    """The dX products of a grouped call with dx_sum, the second of which adds to the first: bit for bit the bf16 sum of what
    the plain calls give (those are compared with the oracle above)."""
    import torch
    import gpu_harness as gh
    from paper_2508_02932_amd import plora
    T, D, K, parts, _, dx = PLANS[case]
    print(f"[case] accumulating {case} {w_layouts}", flush=True)
    lins = [ragged(f"gemm_acc_{case}_{p}", T, D, K, parts, 239 + p) for p in range(2)]
    assert all(plan_of(l, w)[1] == dx for l, w in zip(lins, w_layouts))
    tens = [l.tensors() for l in lins]
    tens[1].x = tens[0].x
    dps = [gh.upload(l, t, w) for l, t, w in zip(lins, tens, w_layouts)]
    for dp in dps:
        gh.forward(dp)
        gh.backward(dp)
    lists = lambda name: [getattr(dp, name) for dp in dps]
    group = plora.Group(lists("desc"))
    ws = torch.empty(plora.plora_group_workspace_bytes(group), dtype=torch.uint8, device="cuda")
    total = torch.full_like(dps[0].dx, float("nan"))
    plora.plora_group_bwd(group, dps[0].x, lists("W"), lists("A"), lists("B"), lists("dy"), lists("h"), None, lists("dA"), lists("dB"), ws,
                          dx_sum=total)
    torch.cuda.synchronize()
    assert torch.equal(total, dps[0].dx + dps[1].dx)


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
    264 -> 648, 35336 tokens: the forward product alone (dX goes to 128-row tiles); 512 -> 512, 32760 tokens: both, one full round."""
    import oracle
    lengths = [300, 7, 90, 0, 61, 4000, 1, 2, 30, 9000, 255, 513, 21000 if tail == 77 else 6000, tail]
    lin = wl.small(f"gemm_256_ragged_{D}", "bf16", D, K, lengths=lengths, seg_adapter=[i % 4 if i % 6 else -1 for i in range(len(lengths))],
                   ranks=[8, 72, 3, 128], scales=[2.0, 1.0, 0.5, 0.25], seed=229)
    run_and_compare(lin, impl=oracle.matmul, w_layout=w_layout)


def test_gemm_splits_cut_to_keep_the_workspace_within_the_scratch_array():
    """A split product whose partial tiles would push the workspace past the scratch array of the call without workspace is
    split less; it still is what the oracle says, and that call gives the same bits."""
    import torch
    import gpu_harness as gh
    import oracle
    from paper_2508_02932_amd import plora
    T, D, K = 1000, 14336, 2048
    cut, whole = (wl.small(f"gemm_small_cut_{n}", "bf16", D, K, lengths=tokens_of(T, n), seg_adapter=list(range(n)), ranks=[r] * n,
                           scales=[1.0] * n, seed=227) for n, r in ((5, 128), (1, 8)))
    assert plan_of(whole)[0] == (128, 4, 0) and plan_of(cut)[0][0] == 128 and 1 < plan_of(cut)[0][1] < 4
    size = plora.plora_workspace_bytes(gh.desc_of(cut))
    assert size <= plora.NOALLOC_SCRATCH_BYTES < size + T * K * 4          # one split more would not fit
    dp, _ = run_and_compare(cut, impl=oracle.matmul)
    y = dp.y.clone()
    dp.y.fill_(float("nan"))
    plora.plora_linear_fwd_noalloc(dp.desc, dp.x, dp.W, dp.A, dp.B, dp.y, dp.h)
    torch.cuda.synchronize()
    assert np.array_equal(gh.to_np(y), gh.to_np(dp.y))
