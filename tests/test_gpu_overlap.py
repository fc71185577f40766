"""Outputs of a backward call in memory that it reads, where plora.h allows it: the launches that hold several products must not
write there while another product still reads.  Every result has the bits of the call with memory of its own."""
import pytest

from paper_2508_02932_amd import plora
from paper_2508_02932_amd import workloads as wl

pytestmark = pytest.mark.gpu


def problem(dtype, D, K, lengths, ranks, seed):
    import gpu_harness as gh
    lin = wl.small(f"overlap_{dtype}_{seed}", dtype, D, K, lengths=lengths, seg_adapter=list(range(len(ranks))), ranks=ranks,
                   scales=[2.0, 0.5, 1.0][:len(ranks)], seed=seed)
    dp = gh.upload(lin, lin.tensors())
    gh.forward(dp)
    return dp


def as_floats(t, shapes):
    """fp32 matrices one behind the other in the memory of t."""
    import torch
    flat, out, at = t.view(-1).view(torch.float32), [], 0
    for a, b in shapes:
        out.append(flat[at:at + a * b].view(a, b))
        at += (a * b + 3) // 4 * 4
    return out


@pytest.mark.parametrize("where", ["x", "h_saved"])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_dx_in_the_memory_of_an_input(dtype, where):
    import torch
    import gpu_harness as gh
    dp = problem(dtype, 520, 752, [300, 477], [20, 7], 463)
    gh.backward(dp)
    torch.cuda.synchronize()
    want = [t.clone() for t in (dp.dx, *dp.dA, *dp.dB)]
    h, dx = dp.h, dp.x
    if where == "h_saved":
        dx = torch.empty_like(dp.x)
        h = dx.view(-1).view(torch.float32)[:dp.h.numel()]
        h.copy_(dp.h)
    for t in (*dp.dA, *dp.dB):
        t.fill_(float("nan"))
    print(f"[case] {dtype} dx in {where}", flush=True)
    plora.plora_linear_bwd(dp.desc, dp.x, dp.W, dp.A, dp.B, dp.dy, h, dx, dp.dA, dp.dB, dp.ws)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(want, (dx, *dp.dA, *dp.dB)))


def test_dA_in_the_memory_of_dy():
    import torch
    import gpu_harness as gh
    dp = problem("bf16", 1024, 520, [300, 410], [64, 40], 467)
    gh.backward(dp)
    torch.cuda.synchronize()
    want = [t.clone() for t in (*dp.dA, *dp.dB)]
    dA = as_floats(dp.dy, [t.shape for t in dp.dA])
    print("[case] dA in dy", flush=True)
    plora.plora_linear_bwd(dp.desc, dp.x, dp.W, dp.A, dp.B, dp.dy, dp.h, None, dA, dp.dB, dp.ws)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(want, (*dA, *dp.dB)))


@pytest.mark.parametrize("dtype,ranks", [("f32", [20, 7]), ("bf16", [128, 100])])
def test_group_gradients_in_the_memory_of_an_earlier_dy(dtype, ranks):
    """(rank 128: the projections are not fused, so the gradients of both are products of one launch)"""
    import torch
    import gpu_harness as gh
    dps = [problem(dtype, 256, K, [300, 477], ranks, 479 + p) for p, K in enumerate((1032, 520))]
    x = dps[0].x
    group = plora.Group([dp.desc for dp in dps])
    ws = torch.empty(plora.plora_group_workspace_bytes(group), dtype=torch.uint8, device="cuda")
    lists = lambda name: [getattr(dp, name) for dp in dps]

    def backward(dA, dB):
        plora.plora_group_bwd(group, x, lists("W"), lists("A"), lists("B"), lists("dy"), None, lists("dx"), dA, dB, ws)
        torch.cuda.synchronize()
        return [t.clone() for t in (*lists("dx"), *[t for g in (*dA, *dB) for t in g])]

    want = backward(lists("dA"), lists("dB"))
    inside = as_floats(dps[0].dy, [t.shape for t in (*dps[1].dA, *dps[1].dB)])
    print(f"[case] group {dtype}", flush=True)
    got = backward([dps[0].dA, inside[:2]], [dps[0].dB, inside[2:]])
    assert all(torch.equal(a, b) for a, b in zip(want, got))
