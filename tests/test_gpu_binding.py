"""The binding's marshalling: what it takes and refuses (None, wrong kinds, hyperparameter tuples), streams, and that the results
of a call do not depend on how its tensors are held (lists, tuples, parameters, views)."""
import numpy as np
import pytest

from paper_2508_02932_amd import workloads as wl

pytestmark = pytest.mark.gpu


def problem():
    import gpu_harness as gh
    lin = wl.small("binding", "bf16", 64, 72, lengths=[20, 30], seg_adapter=[0, 1], ranks=[4, 16], scales=[2.0, 0.5], seed=467)
    return gh.upload(lin, lin.tensors())


@pytest.mark.parametrize("hold", ["tuples", "parameters", "stream"])
def test_same_results(hold):
    import torch
    import gpu_harness as gh
    from paper_2508_02932_amd import plora
    dp = problem()
    gh.forward(dp)
    torch.cuda.synchronize()
    want = dp.y.clone()
    dp.y.fill_(float("nan"))
    A, B, x, stream = dp.A, dp.B, dp.x, None
    if hold == "tuples":
        A, B, x = tuple(A), tuple(B), dp.x.view(dp.x.shape)
    elif hold == "parameters":
        A, B = [torch.nn.Parameter(a, requires_grad=False) for a in A], [torch.nn.Parameter(b, requires_grad=False) for b in B]
    else:
        stream = torch.cuda.Stream()
        stream.wait_stream(torch.cuda.current_stream())
    plora.plora_linear_fwd(dp.desc, x, dp.W, A, B, dp.y, None, dp.ws, stream=stream)
    torch.cuda.synchronize()
    assert torch.equal(dp.y, want)


def test_refusals():
    import torch
    from paper_2508_02932_amd import plora
    dp = problem()
    fwd = lambda x, A, ws: plora.plora_linear_fwd(dp.desc, x, dp.W, A, dp.B, dp.y, dp.h, ws)
    with pytest.raises(plora.PloraError):
        fwd(None, dp.A, dp.ws)
    with pytest.raises(plora.PloraError):
        fwd(dp.x, None, dp.ws)
    with pytest.raises(plora.PloraError):
        fwd(dp.x, dp.A, dp.ws[:256])
    for bad in ([None, dp.A[1]], [dp.A[0], 3]):
        with pytest.raises(AttributeError):
            fwd(dp.x, bad, dp.ws)
    with pytest.raises(AttributeError):
        fwd(dp.x, dp.A, None)
    with pytest.raises(TypeError):
        fwd(dp.x, iter(dp.A), dp.ws)
    side = lambda ts: {"param": ts, **{k: [torch.zeros_like(t, dtype=torch.float32) for t in ts] for k in ("master", "grad", "m", "v")}}
    a, b = side(dp.A), side(dp.B)
    for hp in ((1e-4, 0.9, 0.999, 1e-8, 0.01), (1e-4, 0.9, 0.999, 1e-8, 0.01, 1.0), (1e-4, 0.9, 0.999, 1e-8, 0.01, np.int64(1))):
        with pytest.raises(TypeError):
            plora.plora_adamw_step(dp.desc, a, b, [hp] * 2)
    with pytest.raises(plora.PloraError):
        plora.plora_adamw_step(dp.desc, a, b, [(1e-4, 0.9, 0.999, 1e-8, 0.01, 0)] * 2)          # step counts from 1
    plora.plora_adamw_step(dp.desc, a, b, [(1e-4, 0.9, 0.999, 1e-8, 0.01, 1)] * 2)
    torch.cuda.synchronize()
