"""The forward of a short batch in two launches (shrink and base product side by side, then both sums and the low-rank term): slices at
the edges of segments, rows of the base model alone, more segments than a wave has lanes, ranks that are no multiple of 4 or 16,
contractions and columns that fill no tile, split and unsplit products in either tile height, and the projections of a group in one
launch or apart, against the fp64 oracle and, for groups, bit for bit against the plain calls.  Tolerance as in test_gpu_parity.py."""
import pytest

import oracle
from paper_2508_02932_amd import plora
from paper_2508_02932_amd import workloads as wl
from test_gpu_parity import run_and_compare

pytestmark = pytest.mark.gpu

# d_in, d_out, lengths, owners, ranks, rows of the tiles, split
CASES = {
    "one_token": (72, 136, [1], [0], [1], 64, False),
    "edges": (200, 264, [1, 15, 16, 17, 0, 31, 33, 5, 64, 65], [0, 1, -1, 2, 0, 3, 4, -1, 5, 1], [1, 3, 5, 16, 33, 128], 64, False),
    "split": (4104, 1032, [7, 30, 1, 12], [1, 0, -1, 2], [60, 12, 64], 64, True),
    "many_segments": (1000, 520, [1 + i % 3 for i in range(150)], [i % 5 if i % 3 == 0 else -1 for i in range(150)], [8, 31, 2, 17, 64], 64, False),
    "wide_finish": (320, 4104, [200, 3, 150], [0, -1, 1], [24, 96], 64, False),
    "ring_of_three_split": (4104, 8200, [100, 60, 40], [0, 1, 0], [16, 40], 128, True),
    "128_rows_split": (8200, 4104, [300, 380, 20], [0, 1, -1], [33, 8], 128, True),
    # the finishing launch with four blocks of columns and four steps of rank: 68 KB of LDS
    "wide_rank_117": (328, 5680, [120, 130, 129], [0, 1, 2], [8, 117, 30], 64, False),
    "wide_rank_128": (2056, 4200, [90, 310, 100], [0, -1, 1], [16, 128], 64, False),
    "wide_split": (4200, 7432, [83, 82, 82], [0, 1, 2], [112, 16, 16], 64, True),
}
WIDE = ("128_rows_split", "wide_rank_117", "wide_rank_128", "wide_split")


def finish_workgroups(lengths, K, n=1):
    """Of the finishing launch in its narrow form; above 1024 of them it takes the wide one."""
    return n * sum((v + 15) // 16 for v in lengths) * ((K + 127) // 128)


def counted(call):
    """Brackets of the classes base product, shrink and preparation that a call records."""
    import torch
    plora.plora_set_kernel_timing(True)
    try:
        call()
        torch.cuda.synchronize()
        return tuple(plora.plora_kernel_time(c)[1] for c in (0, 2, 6))
    finally:
        plora.plora_set_kernel_timing(False)


def takes_two_launches(desc, tile_rows, split):
    info = plora.plora_debug_metadata(desc)[0]
    assert info.desc_words <= 896 and info.short_shares[0] > 0
    assert (info.gemm_rows[0], info.gemm_splits[0] > 1, info.gemm_big_tiles[0]) == (tile_rows, split, 0)
    assert split or desc.T * desc.d_out <= 2250000


def problem(name, case, seed=461):
    D, K, lengths, owner, ranks = case[:5]
    return wl.small(f"gemm_short_{name}", "bf16", D, K, lengths=lengths, seg_adapter=owner, ranks=ranks, scales=[2.0, 0.5, 1.25, 1.0, 3.0, 4.0][:len(ranks)],
                    seed=seed)


@pytest.mark.parametrize("w_layout", [0, 1])
@pytest.mark.parametrize("save_h", [True, False])
@pytest.mark.parametrize("case", sorted(CASES))
def test_two_launches(case, save_h, w_layout):
    import gpu_harness as gh
    lin = problem(case, CASES[case])
    takes_two_launches(gh.desc_of(lin, w_layout), *CASES[case][5:])
    D, K, lengths = CASES[case][:3]
    assert (finish_workgroups(lengths, K) > 1024) == (case in WIDE)
    dp, _ = run_and_compare(lin, impl=oracle.matmul, save_h=save_h, w_layout=w_layout)
    assert counted(lambda: gh.forward(dp, save_h)) == (1, 0, 0)        # shrink, preparation and product in one bracket


@pytest.mark.parametrize("w_layouts", [(0, 0, 0), (1, 0, 1)])
def test_group_is_bitwise_the_plain_calls(w_layouts):
    """Three projections of one input, the last in tiles of another height and so in launches of its own."""
    import torch
    import gpu_harness as gh
    lengths, owner, ranks = [100, 3, 60, 37], [0, -1, 1, 0], [20, 64]
    lins = [problem(f"group_{p}", (4104, K, lengths, owner, ranks), 467 + p) for p, K in enumerate((520, 264, 8200))]
    tens = [l.tensors() for l in lins]
    for t in tens[1:]:
        t.x = tens[0].x
    dps = [gh.upload(l, t, w) for l, t, w in zip(lins, tens, w_layouts)]
    for dp, rows in zip(dps, (64, 64, 128)):
        takes_two_launches(dp.desc, rows, True)
        gh.forward(dp)
    want = [(dp.y.clone(), dp.h.clone()) for dp in dps]
    for dp in dps:
        dp.y.fill_(float("nan")); dp.h.fill_(float("nan"))
    group_is_the_plain_calls(dps, want, (1, 0, 0))


def group_is_the_plain_calls(dps, want, brackets):
    import torch
    lists = lambda name: [getattr(dp, name) for dp in dps]
    group = plora.Group(lists("desc"))
    ws = torch.empty(plora.plora_group_workspace_bytes(group), dtype=torch.uint8, device="cuda")
    assert counted(lambda: plora.plora_group_fwd(group, dps[0].x, lists("W"), lists("A"), lists("B"), lists("y"), lists("h"), ws)) == brackets
    for dp, (y, h) in zip(dps, want):
        n = plora.plora_h_elems(dp.desc)
        assert torch.equal(dp.y, y) and torch.equal(dp.h[:n], h[:n])


@pytest.mark.parametrize("w_layout", [0, 1])
def test_group_with_the_wide_finish(w_layout):
    """Two projections whose plain calls finish in the narrow form and together in the wide one, at four steps of rank (68 KB of LDS)."""
    import gpu_harness as gh
    D, lengths, owner, ranks = 328, [120, 130, 129], [0, 1, 2], [8, 117, 30]
    lins = [problem(f"group_wide_{p}", (D, K, lengths, owner, ranks), 503 + p) for p, K in enumerate((2808, 2200))]
    tens = [l.tensors() for l in lins]
    tens[1].x = tens[0].x
    dps = [gh.upload(l, t, w_layout) for l, t in zip(lins, tens)]
    for dp in dps:
        takes_two_launches(dp.desc, 64, False)
        assert finish_workgroups(lengths, dp.desc.d_out) <= 1024
        gh.forward(dp)
    assert finish_workgroups(lengths, 2808, 2) > 1024
    want = [(dp.y.clone(), dp.h.clone()) for dp in dps]
    for dp in dps:
        dp.y.fill_(float("nan")); dp.h.fill_(float("nan"))
    group_is_the_plain_calls(dps, want, (1, 0, 0))


MIXED = {   # tokens, d_in, widths: the first projection does not take the two launches; brackets of products, shrinks, preparations
    "few_sums": (461, 1024, (5408, 1352, 1352), (2, 1, 1)),             # the others do, 1.25 M sums
    "many_sums": (1240, 864, (4904, 1224, 1224), (3, 1, 1)),            # 3.0 M: they share the group's steps
    "split": (432, 4736, (8944, 2232, 2232), (2, 1, 1)),                # split anyway
}


@pytest.mark.parametrize("w_layout", [0, 1])
@pytest.mark.parametrize("case", sorted(MIXED))
def test_group_of_both_kinds(case, w_layout):
    """Projections in two launches beside one that is not, and the same in the group's own steps: the bits of the plain calls."""
    import gpu_harness as gh
    T, D, widths, brackets = MIXED[case]
    lengths, owner, ranks = [T // 3, 5, T - T // 3 - 5], [0, -1, 1], [30, 8]
    lins = [problem(f"group_{case}_{p}", (D, K, lengths, owner, ranks), 509 + p) for p, K in enumerate(widths)]
    tens = [l.tensors() for l in lins]
    for t in tens[1:]:
        t.x = tens[0].x
    dps = [gh.upload(l, t, w_layout) for l, t in zip(lins, tens)]
    for dp, plain in zip(dps, ((1, 0, 1), (1, 0, 0), (1, 0, 0))):
        assert counted(lambda: gh.forward(dp)) == plain
    want = [(dp.y.clone(), dp.h.clone()) for dp in dps]
    for dp in dps:
        dp.y.fill_(float("nan")); dp.h.fill_(float("nan"))
    group_is_the_plain_calls(dps, want, brackets)
