"""A backward pass whose activation was not saved: the shrink and dH run in one launch where neither is short and there is room for
both sets of partial tiles, and every result has the bits of the pass that was given the saved activation."""
import numpy as np
import pytest

import oracle
from oracle import nf4
from paper_2508_02932_amd import plora
from paper_2508_02932_amd import workloads as wl
from test_gpu_parity import TOL, run_and_compare
from util import make_problem, scaled_err

pytestmark = pytest.mark.gpu

MANY = [1 + 37 * i % 160 for i in range(80)]      # above 64 blocks of rows: not short
CASES = {
    "wide_in": (2504, 72, MANY, [1 + 7 * i % 40 for i in range(80)]),
    "wide_out": (72, 2504, MANY, [1 + 7 * i % 40 for i in range(80)]),
    "both_split": (1032, 2056, MANY, [16] * 80),
    "few_rows": (4104, 4096, [1] * 70 + [129], [3, 128] + [1] * 69),
    "one_launch_wide_in": (8192, 512, MANY, [1 + 7 * i % 16 for i in range(80)]),
    "one_launch_wide_out": (512, 8200, MANY, [1 + 7 * i % 16 for i in range(80)]),
}


def one_launch(desc):
    """Whether dH's partial tiles have room beside the shrink's (so that both products are entries of one launch)."""
    info = plora.plora_debug_metadata(desc)[0]
    return info.dh_splits * info.n_blocks * 128 * info.max_r16 * 4 <= info.ws_total - 256 - info.ws_wpart, list(info.short_shares)


@pytest.mark.parametrize("w_layout", [0, 1])
@pytest.mark.parametrize("case", sorted(CASES))
def test_recomputed_is_bitwise_the_saved(case, w_layout):
    import torch
    import gpu_harness as gh
    D, K, lengths, ranks = CASES[case]
    lin = wl.small(f"recomputed_{case}", "bf16", D, K, lengths=lengths, seg_adapter=list(range(len(ranks))), ranks=ranks,
                   scales=[1.0 + i % 3 for i in range(len(ranks))], seed=457)
    assert one_launch(gh.desc_of(lin, w_layout)) == (case.startswith("one_launch"), [0, 0])
    dp, _ = run_and_compare(lin, impl=oracle.matmul, w_layout=w_layout)
    saved = [t.clone() for t in (dp.dx, *dp.dA, *dp.dB)]
    for t in (dp.dx, *dp.dA, *dp.dB):
        t.fill_(float("nan"))
    gh.backward(dp, use_saved_h=False)
    torch.cuda.synchronize()
    gh.check_guards(dp)
    assert all(torch.equal(a, b) for a, b in zip(saved, (dp.dx, *dp.dA, *dp.dB))), case


@pytest.mark.parametrize("w_layout", [0, 1])
@pytest.mark.parametrize("D,K,lengths,ranks", [(1024, 2048, [300, 212], [64, 16]), (1032, 4104, [333, 0, 190], [16, 3, 9])])
def test_nf4_recomputed_is_bitwise_the_saved(D, K, lengths, ranks, w_layout):
    """Over an NF4 weight no product takes the routine for short batches, so few rows share a launch as well."""
    import torch
    import gpu_harness as gh
    lin = wl.small("recomputed_nf4", "bf16", D, K, lengths=lengths, seg_adapter=list(range(len(ranks))), ranks=ranks,
                   scales=[2.0, 0.5, 1.0][:len(ranks)], seed=463)
    t = lin.tensors()
    W_mem = np.ascontiguousarray(t.W.T if w_layout else t.W)
    codes, absmax = nf4.quantize(W_mem.ravel())
    W_deq = nf4.dequantize(codes, absmax, W_mem.size, "bf16").reshape(W_mem.shape)
    t.W = np.ascontiguousarray(W_deq.T if w_layout else W_deq)
    dp = gh.upload(lin, t, w_layout)
    assert one_launch(dp.desc)[0]
    guards: list = []
    ws = gh.guarded((plora.plora_nf4_workspace_bytes(dp.desc),), torch.uint8, None, guards, "workspace")
    c, a = torch.from_numpy(codes).cuda(), torch.from_numpy(absmax).cuda()
    plora.plora_linear_fwd_nf4(dp.desc, dp.x, c, a, dp.A, dp.B, dp.y, dp.h, ws)
    got = []
    for h in (dp.h, None):
        for out in (dp.dx, *dp.dA, *dp.dB):
            out.fill_(float("nan"))
        print(f"[case] nf4 backward, saved activation: {h is not None}", flush=True)
        plora.plora_linear_bwd_nf4(dp.desc, dp.x, c, a, dp.A, dp.B, dp.dy, h, dp.dx, dp.dA, dp.dB, ws)
        torch.cuda.synchronize()
        got.append([out.clone() for out in (dp.dx, *dp.dA, *dp.dB)])
    gh.check_guards(dp)
    for name, base, nbytes in guards:
        assert bool((base[:gh.GUARD_BYTES] == gh.GUARD_BYTE).all()) and bool((base[gh.GUARD_BYTES + nbytes:] == gh.GUARD_BYTE).all()), name
    assert all(torch.equal(u, v) for u, v in zip(*got))
    dx_o, _, dA_o, dB_o = oracle.matmul.backward(make_problem(oracle, lin, t), t.dy)
    errs = [scaled_err(gh.to_np(u), v) for u, v in zip(got[1], (dx_o, *dA_o, *dB_o))]
    assert all(np.isfinite(e) and e <= TOL["bf16"] for e in errs), errs
