"""dX in small tiles beside dB and dA, in one launch: split and unsplit products beside split and whole token walks, either tile
height, both weight orders, against the fp64 oracle and bit for bit against the same call with dx in the memory of x, which runs
one product after the other.  Tolerance as in test_gpu_parity.py."""
import pytest

import oracle
from paper_2508_02932_amd import plora
from paper_2508_02932_amd import workloads as wl
from test_gpu_parity import run_and_compare

pytestmark = pytest.mark.gpu

CASES = {
    # d_in, d_out, lengths, ranks, rows of the tiles, splits of dX, of dA, of dB
    "one_token": (72, 136, [1], [3], 64, 1, 1, 1),
    "all_whole": (264, 520, [100, 31, 64], [16, 5, 100], 64, 1, 1, 1),
    "split_dx": (520, 4104, [90, 33], [16, 9], 64, 11, 1, 1),
    "split_walks": (1032, 392, [900, 460], [24, 8], 64, 1, 2, 2),
    "all_split": (520, 4104, [700, 460], [24, 8], 64, 5, 2, 2),
    "128_rows": (4104, 4104, [500, 523], [16, 40], 128, 1, 1, 1),
    "ring_of_three": (8200, 4104, [100, 60, 40], [16, 40, 8], 128, 3, 1, 1),
}


def problem(case):
    D, K, lengths, ranks = CASES[case][:4]
    return wl.small(f"grads_{case}", "bf16", D, K, lengths=lengths, seg_adapter=list(range(len(ranks))), ranks=ranks, scales=[2.0, 0.5, 1.25][:len(ranks)],
                    seed=479)


@pytest.mark.parametrize("w_layout", [0, 1])
@pytest.mark.parametrize("case", sorted(CASES))
def test_grads_and_dx(case, w_layout):
    import torch
    import gpu_harness as gh
    lin = problem(case)
    info = plora.plora_debug_metadata(gh.desc_of(lin, w_layout))[0]
    assert (info.gemm_rows[1], info.gemm_splits[1], info.da_splits, info.db_splits) == CASES[case][4:] and info.gemm_big_tiles[1] == 0
    dp, _ = run_and_compare(lin, impl=oracle.matmul, w_layout=w_layout)
    want = [t.clone() for t in (dp.dx, *dp.dA, *dp.dB)]
    for dx, launches in ((dp.dx, 0), (dp.x, 1)):             # launches of the weight gradients alone
        for t in (*dp.dA, *dp.dB):
            t.fill_(float("nan"))
        plora.plora_set_kernel_timing(True)
        try:
            plora.plora_linear_bwd(dp.desc, dp.x, dp.W, dp.A, dp.B, dp.dy, dp.h, dx, dp.dA, dp.dB, dp.ws)
            torch.cuda.synchronize()
            assert plora.plora_kernel_time(4)[1] == launches
        finally:
            plora.plora_set_kernel_timing(False)
        assert all(torch.equal(a, b) for a, b in zip(want, (dx, *dp.dA, *dp.dB)))


@pytest.mark.parametrize("total", [False, True])
@pytest.mark.parametrize("w_layout", [0, 1])
def test_first_projection_of_a_group(w_layout, total):
    """dX of the first projection beside dB of all, the second's behind it: the bits of the plain calls and of their sum."""
    import torch
    import gpu_harness as gh
    D, lengths, ranks = 520, [700, 460], [24, 8]
    lins = [wl.small(f"grads_group_{p}", "bf16", D, K, lengths=lengths, seg_adapter=[0, 1], ranks=ranks, scales=[2.0, 0.5], seed=491 + p)
            for p, K in enumerate((4104, 392))]
    tens = [l.tensors() for l in lins]
    tens[1].x = tens[0].x
    dps = [gh.upload(l, t, w_layout) for l, t in zip(lins, tens)]
    for dp in dps:
        gh.forward(dp)
        gh.backward(dp)
    want = [[t.clone() for t in (dp.dx, *dp.dA, *dp.dB)] for dp in dps]
    for dp in dps:
        for t in (dp.dx, *dp.dA, *dp.dB):
            t.fill_(float("nan"))
    lists = lambda name: [getattr(dp, name) for dp in dps]
    group = plora.Group(lists("desc"))
    ws = torch.empty(plora.plora_group_workspace_bytes(group), dtype=torch.uint8, device="cuda")
    out = torch.full_like(dps[0].dx, float("nan"))
    plora.plora_set_kernel_timing(True)
    try:
        plora.plora_group_bwd(group, dps[0].x, lists("W"), lists("A"), lists("B"), lists("dy"), lists("h"), None if total else lists("dx"),
                              lists("dA"), lists("dB"), ws, dx_sum=out if total else None)
        torch.cuda.synchronize()
        assert plora.plora_kernel_time(4)[1] == 0
    finally:
        plora.plora_set_kernel_timing(False)
    if total:
        assert torch.equal(out, want[0][0] + want[1][0])
    for dp, w in zip(dps, want):
        if not total:
            assert torch.equal(dp.dx, w[0])
        assert all(torch.equal(a, b) for a, b in zip((*dp.dB,), w[1 + len(ranks):]))
        # the fused pass may split the token walk otherwise: fp32 sums over 700 tokens in another order, sqrt(700) 2^-24 = 1.6e-6 of them
        for a, b in zip(dp.dA, w[1:]):
            assert (a - b).abs().max() <= 1e-5 * b.abs().max()
