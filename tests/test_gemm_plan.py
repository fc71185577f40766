"""Where the 256 x 256 tiles of the base GEMM take a split contraction and where small tiles do (host only): a handful of tokens, many
extension steps, and a product that small tiles would run together with a short shrink stay in small tiles."""
import numpy as np
import pytest

from paper_2508_02932_amd import plora


def plan(T, D, K, ranks, w_layout):
    n = len(ranks)
    lengths = [T // n + (i < T % n) for i in range(n)]
    d = plora.Desc(T, D, K, np.concatenate([[0], np.cumsum(lengths)]), np.arange(n), np.array(ranks), np.ones(n), plora.PLORA_BF16, w_layout)
    info, _, _ = plora.plora_debug_metadata(d)
    return [(info.gemm_rows[i], info.gemm_splits[i], info.gemm_big_tiles[i]) for i in range(2)]


SMALL = {   # T, D, K, ranks: the forward product in small tiles
    "one_token": (1, 8192, 8192, [16]),
    "64_tokens": (64, 8192, 8192, [16]),
    "few_tokens_ragged_rows": (26, 6800, 8064, [80] * 7),
    "eight_of_rank_64": (80, 8192, 8192, [64] * 8),
    "sixteen_of_rank_32": (128, 8192, 8192, [32] * 16),
    "two_steps_a_segment": (256, 14336, 8192, [100] * 16),
    "many_segments": (512, 8192, 14336, [16] * 128),
    "two_launches_with_the_shrink": (640, 8192, 4096, [16]),
    "two_launches_two_row_tiles": (330, 7168, 7168, [16]),
}
SPLIT = {   # ... in 256 x 256 tiles, and the parts of it
    "65_tokens": (65, 8640, 17408, [16], 3),
    "rows_that_share_lines": (72, 11464, 16824, [16], 3),
    "six_steps": (72, 11456, 16832, [16] * 6, 3),
    "two_row_tiles": (512, 8192, 8192, [16], 3),
    "seven_row_tiles": (1500, 8200, 2040, [32] * 8, 4),
    "many_segments_in_many_row_tiles": (3000, 16384, 1024, [8] * 256, 4),
}


@pytest.mark.parametrize("w_layout", [0, 1])
@pytest.mark.parametrize("case", sorted(SMALL))
def test_small_tiles(case, w_layout):
    (rows, _, big), _ = plan(*SMALL[case], w_layout)
    assert rows in (64, 128) and big == 0


@pytest.mark.parametrize("w_layout", [0, 1])
@pytest.mark.parametrize("case", sorted(SPLIT))
def test_split_256_tiles(case, w_layout):
    T, D, K, ranks, parts = SPLIT[case]
    assert plan(T, D, K, ranks, w_layout)[0] == (0, parts, (T + 255) // 256)


def test_the_gradient_of_x_follows_the_same_lines():
    """Its contraction and columns are the forward's the other way round; it never runs in two launches with the shrink."""
    for w_layout in (0, 1):
        assert plan(8192, 8192, 8192, [16], w_layout)[1][0] == 0
        assert plan(64, 8192, 8192, [16], w_layout)[1][0] == 64
        assert plan(640, 4096, 8192, [16], w_layout)[1] == (0, 5, 3)
    # ten extension steps: 2.5 us for each behind the sixth where the contraction runs over W's rows, 1 us where along them
    assert plan(128, 9448, 13040, [16] * 10, 0)[1] == (0, 6, 1) and plan(128, 9448, 13040, [16] * 10, 1)[1][0] == 64
