"""The workspace of grouped calls holds the partial tiles of every fused pass that a call can ask for.  A backward call fuses
dA over the projections that want weight gradients, which may be any two or more of a cell, and a smaller fused rank can mean
more splits of the token walk.  Host only: a pass over projections of ranks r_p is split as a plain call of rank sum(r16_p)
on the same tokens is, so plora_debug_metadata of such a description says what the pass needs."""
import itertools

import numpy as np
import pytest

from paper_2508_02932_amd import plora


def pad(v, a):
    return (v + a - 1) // a * a


def desc(T, D, K, lengths, owner, ranks):
    return plora.Desc(T, D, K, np.concatenate([[0], np.cumsum(lengths)]), np.array(owner), np.array(ranks),
                      np.ones(len(ranks)), plora.PLORA_BF16)


def check(D, Ks, lengths, owner, ranks):
    """ranks[p][k]: rank of adapter k in projection p."""
    T = sum(lengths)
    descs = [desc(T, D, K, lengths, owner, r) for K, r in zip(Ks, ranks)]
    room = plora.plora_group_workspace_bytes(plora.Group(descs)) - sum(pad(plora.plora_workspace_bytes(d), 256) for d in descs)
    padded = [[pad(v, 16) for v in r] for r in ranks]
    fused = lambda members: [sum(padded[p][k] for p in members) for k in range(len(ranks[0]))]
    cells, cell = [], []
    for p in range(len(Ks)):                     # consecutive projections whose padded ranks sum to 128 at most
        if cell and max(fused(cell + [p])) > 128:
            cells.append(cell)
            cell = []
        cell.append(p)
    splits = set()
    for cell in cells + [cell]:
        for n in range(2, len(cell) + 1):
            for members in itertools.combinations(cell, n):
                f = fused(members)
                info, _, _ = plora.plora_debug_metadata(desc(T, D, 64, lengths, owner, f))
                splits.add(info.da_splits)
                if info.da_splits > 1:
                    assert info.da_splits * sum(f) * D * 4 <= room, (members, info.da_splits)
    return splits


def test_projections_left_out_of_the_fused_dA_pass():
    # all three: 96 rank rows, one split; two of them: 64 rows, two splits, 16.8 MB of partial tiles
    assert check(8192, [64] * 3, [1250] * 4, list(range(4)), [[32] * 4] * 3) == {1, 2}


@pytest.mark.parametrize("seed", range(40))
def test_generated_groups(seed):
    rng = np.random.default_rng(seed)
    n, n_ad = int(rng.integers(2, 5)), int(rng.integers(1, 9))
    ranks = [[int(v) for v in rng.integers(1, 129 // n, size=n_ad)] for _ in range(n)]
    lengths = [int(v) for v in rng.integers(0, 3000, size=n_ad)]
    check(8 * int(rng.integers(64, 1200)), [int(v) * 8 for v in rng.integers(8, 64, size=n)], lengths, list(range(n_ad)), ranks)
