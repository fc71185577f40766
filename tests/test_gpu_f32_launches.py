"""The fp32 path's launches: low-rank products beside the preparation and, behind a long description, in a launch of their own; more
segments in a row tile than a wave looks up at once; weight gradients with and without the gradient of x in the launch."""
import numpy as np
import pytest

import oracle
from paper_2508_02932_amd import workloads as wl
from test_gpu_parity import TOL, run_and_compare
from util import make_problem, scaled_err

pytestmark = pytest.mark.gpu

CASES = {
    "many_segments_in_a_tile": (36, 40, [1 + i % 3 for i in range(150)], [i % 5 - 1 for i in range(150)], [1, 7, 16, 33]),
    "long_description": (40, 24, [2 + i % 9 for i in range(95)], list(range(95)), [1 + 7 * i % 40 for i in range(95)]),
    "edges": (33, 65, [1, 31, 32, 33, 0, 100], [0, 1, 2, 0, 1, -1], [1, 17, 128]),
}


@pytest.mark.parametrize("w_layout", [0, 1])
@pytest.mark.parametrize("save_h", [True, False])
@pytest.mark.parametrize("case", sorted(CASES))
def test_f32(case, save_h, w_layout):
    D, K, lengths, owner, ranks = CASES[case]
    lin = wl.small(f"f32_{case}", "f32", D, K, lengths=lengths, seg_adapter=owner, ranks=ranks, scales=[1.0 + 0.5 * (i % 4) for i in range(len(ranks))],
                   seed=457)
    run_and_compare(lin, impl=oracle.matmul, save_h=save_h, w_layout=w_layout)


@pytest.mark.parametrize("want_dx,want_w", [(True, False), (False, True)])
def test_one_kind_of_gradient(want_dx, want_w):
    import torch
    import gpu_harness as gh
    from paper_2508_02932_amd import plora
    D, K, lengths, owner, ranks = CASES["edges"]
    lin = wl.small("f32_one_kind", "f32", D, K, lengths=lengths, seg_adapter=owner, ranks=ranks, scales=[2.0, 0.5, 1.0], seed=461)
    t = lin.tensors()
    dx_o, _, dA_o, dB_o = oracle.matmul.backward(make_problem(oracle, lin, t), t.dy)
    dp = gh.upload(lin, t)
    gh.forward(dp)
    plora.plora_linear_bwd(dp.desc, dp.x, dp.W, dp.A, dp.B, dp.dy, dp.h, dp.dx if want_dx else None, dp.dA if want_w else None,
                           dp.dB if want_w else None, dp.ws)
    torch.cuda.synchronize()
    gh.check_guards(dp)
    errs = [scaled_err(gh.to_np(dp.dx), dx_o)] if want_dx else []
    for k in range(len(ranks) if want_w else 0):
        errs += [scaled_err(gh.to_np(dp.dA[k]), dA_o[k]), scaled_err(gh.to_np(dp.dB[k]), dB_o[k])]
    assert all(np.isfinite(e) and e <= TOL["f32"] for e in errs), errs
