"""How a call's launch plan is kept within the scratch array of plora_linear_fwd_noalloc (host only)."""
import numpy as np
import pytest

from paper_2508_02932_amd import plora

LIMIT = plora.NOALLOC_SCRATCH_BYTES


def desc(D, K, lengths, owner, ranks, w_layout=0, dtype=plora.PLORA_BF16):
    return plora.Desc(sum(lengths), D, K, np.concatenate([[0], np.cumsum(lengths)]), np.array(owner), np.array(ranks),
                      np.ones(len(ranks)), dtype, w_layout)


def skinny_rule(n_blocks, C):
    """Splits of the contraction that the token blocks ask for: three workgroups per compute unit and eight stages of 64 per
    split, up to 32 blocks one workgroup per compute unit and four stages."""
    stages = (C + 63) // 64
    coarse = max(1, min(8, -(-768 // n_blocks), stages // 8))
    return max(coarse, min(32, 256 // n_blocks, stages // 4))


@pytest.mark.parametrize("w_layout", [0, 1])
@pytest.mark.parametrize("D,K,T,n", [(4096, 28672, 1228, 8), (8192, 28672, 573, 3), (4096, 28672, 512, 1), (28672, 4096, 700, 2)])
def test_the_skinny_passes_keep_their_splits_where_only_the_gemm_outgrows(D, K, T, n, w_layout):
    """The GEMM's partial tiles lie over the skinny ones and reach further here: cutting the skinny splits gains no room."""
    lengths = [T // n + (i < T % n) for i in range(n)]
    info, _, _ = plora.plora_debug_metadata(desc(D, K, lengths, range(n), [8] * n, w_layout))
    assert info.ws_total <= LIMIT
    assert (info.shrink_splits, info.dh_splits) == (skinny_rule(info.n_blocks, D), skinny_rule(info.n_blocks, K))


def test_the_skinny_passes_are_cut_only_as_far_as_needed():
    info, _, _ = plora.plora_debug_metadata(desc(8192, 64, [150] * 4 + [0] * 24, range(28), [64] * 28))
    assert info.ws_total <= LIMIT and 8 < info.shrink_splits < 32
    per_split = info.n_blocks * 128 * 64 * 4
    assert info.ws_total + per_split > LIMIT


def size_without_records(d):
    """What decides whether plora_linear_fwd_noalloc takes a description: its workspace with eight skinny splits, no split
    GEMM, and tables without the records that the bf16 kernels start from."""
    al = lambda v, a=256: (v + a - 1) // a * a
    info, tab, _ = plora.plora_debug_metadata(d)
    bf = d.dtype == plora.PLORA_BF16
    e2 = 2 if bf else 0
    own = [g for g in tab["seg"] if g["adapter"] >= 0]
    o = 1024 + al(al(int(info.off_tile_order) + 4 * int(info.n_tiles), 64))
    o += al(4 * int(info.desc_words) if info.desc_words > 896 else 0)
    o += al(sum(int(a["r16"]) for a in tab["ad"]) * d.d_in * e2)
    o += al(sum(int(a["rp"]) for a in tab["ad"]) * (d.d_out if d.w_layout else d.d_in) * e2)
    o += al(sum(int(g["row1"] - g["row0"]) * int(g["rp"]) for g in own) * e2)
    o += 2 * al(sum(int(g["r16"]) * int(g["lp"]) for g in own) * e2)
    o += al(4 * int(info.h_elems)) * (1 if bf else 2)
    if bf:
        o += al(8 * int(info.n_blocks) * 128 * int(info.max_r16) * 4)
        o += al(max([s * int(info.r16_total) * w * 4 for s, w in ((info.da_splits, d.d_in), (info.db_splits, d.d_out)) if s > 1] + [0]))
    return o + 256


FAMILIES = {
    # D, K, dtype, ranks, segments of T tokens
    "few_adapters": (512, 512, plora.PLORA_BF16, [16] * 4, lambda T: ([T // 4] * 3 + [T - T // 4 * 3], [0, 1, 2, 3])),
    "f32": (8, 16, plora.PLORA_F32, [1], lambda T: ([T], [0])),
    "f32_ranks": (64, 64, plora.PLORA_F32, [8, 3], lambda T: ([T // 3, T - T // 3], [1, 0])),
    "no_tokens_with_an_adapter": (1184, 64, plora.PLORA_BF16, [64] * 220, lambda T: ([T], [-1])),
    "many_adapters_one_block": (808, 64, plora.PLORA_BF16, [64] * 256, lambda T: ([T, 3], [-1, 7])),
    "eight_splits": (8192, 512, plora.PLORA_BF16, [64] * 29, lambda T: ([T - 5, 5], [3, 4])),
}


@pytest.mark.parametrize("w_layout", [0, 1])
@pytest.mark.parametrize("family", sorted(FAMILIES))
def test_the_records_refuse_nothing_that_fitted_the_scratch_array(family, w_layout):
    """Around the number of tokens at which a description stops fitting: at and below it the workspace is within the scratch
    array, above it is not, so that what was accepted is accepted and what was refused is refused."""
    D, K, dtype, ranks, cut = FAMILIES[family]
    make = lambda T: desc(D, K, *cut(T), ranks, w_layout, dtype)
    lo, hi = 16, 4000000
    assert size_without_records(make(lo)) <= LIMIT
    if size_without_records(make(hi)) <= LIMIT:
        hi = lo
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (mid, hi) if size_without_records(make(mid)) <= LIMIT else (lo, mid)
    for T in (max(16, lo - 700), max(16, lo - 100), max(16, lo - 1), lo, lo + 1, lo + 200):
        d = make(T)
        assert (plora.plora_workspace_bytes(d) <= LIMIT) == (size_without_records(d) <= LIMIT), T


def test_the_scratch_array_takes_a_description_within_100_kb_of_its_size():
    """85400 tokens of four adapters of rank 16: 67 061 504 bytes without the records, 67 108 864 is the limit."""
    d = desc(512, 512, [21350] * 4, range(4), [16] * 4)
    assert size_without_records(d) == 67061504 and plora.plora_workspace_bytes(d) <= LIMIT


@pytest.mark.parametrize("w_layout", [0, 1])
@pytest.mark.parametrize("D,K,T,dense_split", [(2816, 6528, 2554, 2), (768, 7296, 6144, 3), (768, 2048, 1024, 1)])
def test_the_nf4_calls_have_no_room_for_partial_tiles_of_the_dense_ones(D, K, T, dense_split, w_layout):
    """Their product of an expanded weight is not split here, and their forward never takes the two launches of a short batch: behind
    the tables and copies there are the partial tiles of shrink, dH and the weight gradients and nothing else.  (The dense calls: a dX in parts,
    or a shrink's sums and an unsplit product's.)"""
    d = desc(D, K, [T // 2, T - T // 2], [0, 1], [16, 8], w_layout)
    info, _, _ = plora.plora_debug_metadata(d)
    assert info.gemm_splits[1] == dense_split
    grads = max([s * int(info.r16_total) * w * 4 for s, w in ((info.da_splits, D), (info.db_splits, K)) if s > 1] + [0])
    dh = int(info.dh_splits) * int(info.n_blocks) * 128 * int(info.max_r16) * 4
    most = int(info.ws_wpart) + max(grads, dh) + 1024
    assert plora.lib().plora_nf4_workspace_bytes(d.ref) - 2 * D * K <= most < int(info.ws_total)
