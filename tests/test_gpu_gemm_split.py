"""The 256 x 256 tiles of the base GEMM with the contraction split over workgroups: partial last row tiles, column tiles and steps, row
tiles with one, two and many segments (the extension belongs to the first part, whatever its share of the steps), both forms of
the weight, and the accumulating sum of a grouped call, against the fp64 oracle.  Plans and tolerance as in test_gpu_gemm_small.py."""
import pytest

import test_gpu_gemm_small as small
from test_gpu_parity import run_and_compare

pytestmark = pytest.mark.gpu

PLANS = {
    # T, D, K, segments, plan of the forward product, plan of dX
    "three_parts": (2000, 8200, 2040, 3, (0, 3, 8), (64, 1, 7)),
    "four_parts": (900, 8200, 3064, 5, (0, 4, 4), (64, 1, 0)),
    "five_parts": (520, 11272, 4104, 5, (0, 5, 3), (128, 1, 0)),
    "six_parts": (400, 14344, 4104, 5, (0, 6, 2), (0, 2, 2)),
    "six_parts_dx": (400, 4104, 14344, 2, (0, 2, 2), (0, 6, 2)),
    "dx": (3900, 1016, 6008, 9, (0, 1, 16), (0, 3, 16)),                    # four parts would push the workspace past the scratch array
    "many_segments": (2000, 8200, 2040, 295, (0, 3, 8), (64, 1, 7)),      # 49 extension steps in a row tile, 44 steps in a part
    "short_segments": (88, 9984, 4480, 29, (64, 4, 0), (64, 2, 0)),       # so many that small tiles, which share them, are faster
}


@pytest.mark.parametrize("w_layout", [0, 1])
@pytest.mark.parametrize("case", sorted(PLANS))
def test_split(case, w_layout):
    import oracle
    T, D, K, parts, fwd, dx = PLANS[case]
    lin = small.ragged(f"gemm_split_{case}", T, D, K, parts, 241)
    assert small.plan_of(lin, w_layout) == [fwd, dx]
    run_and_compare(lin, impl=oracle.matmul, w_layout=w_layout)


@pytest.mark.parametrize("w_layouts", [(0, 0), (1, 1)])
def test_split_accumulating(monkeypatch, w_layouts):
    monkeypatch.setitem(small.PLANS, "dx", PLANS["dx"])
    small.test_planned_tiles_accumulating("dx", w_layouts)
