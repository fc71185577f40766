"""The calls under HIP graph capture: a forward and a backward call recorded once and replayed several times, with
eager work of the same program between the replays, must reproduce the eager results bit for bit every time (the
calls only enqueue kernels - no synchronisation, no memset, no host-side allocation - and the packing description
travels as a kernel argument, so a replay needs nothing from the host)."""
import numpy as np
import pytest

from paper_2508_02932_amd import plora
from paper_2508_02932_amd import workloads as wl
from test_gpu_parity import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["fused", "lora_only"])
def test_capture_and_replay(mode):
    import torch
    import gpu_harness as gh
    lin = wl.small(f"graph_{mode}", "bf16", 328, 264, lengths=[130, 0, 257, 64, 249, 1, 300],
                   seg_adapter=[1, 0, 2, -1, 1, 0, 2], ranks=[8, 24, 72], scales=[2.0, 0.5, 1.25], seed=541)
    t = lin.tensors()
    lora_only = mode == "lora_only"
    dp = gh.upload(lin, t, lora_only=lora_only)
    base_y = torch.randn_like(dp.y)
    base_dx = torch.randn_like(dp.dx)

    def step():
        if lora_only:
            dp.y.copy_(base_y)
            dp.dx.copy_(base_dx)
            gh.lora_forward(dp)
            gh.lora_backward(dp)
        else:
            gh.forward(dp)
            gh.backward(dp)

    def snapshot():
        torch.cuda.synchronize()
        return [dp.y.clone(), dp.dx.clone(), dp.h.clone()] + [a.clone() for a in dp.dA] + [b.clone() for b in dp.dB]

    step()                                         # eager: also the one-time set-up of the library on this device
    want = snapshot()
    say(f"[case] graph capture {mode}")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        step()                                     # warm-up on the capture stream
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=side):
            step()
    torch.cuda.synchronize()
    for rep in range(4):
        # eager work of the same program between replays: scribble over the outputs and the workspace
        for buf in (dp.y, dp.dx, dp.h, *dp.dA, *dp.dB):
            buf.fill_(float("nan"))
        dp.ws.fill_(0xAB)
        torch.cuda.synchronize()
        graph.replay()
        got = snapshot()
        for a, b in zip(got, want):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), f"replay {rep} differs from the eager run"
    gh.check_guards(dp)


def test_capture_and_replay_grouped():
    """The grouped calls (three projections on one x, one fused pass each way) under capture: as above."""
    import torch
    import gpu_harness as gh
    lengths, seg_adapter = [130, 0, 257, 64, 249], [1, 0, 2, -1, 1]
    lins = [wl.small(f"graph_group_p{p}", "bf16", 328, K, lengths, seg_adapter, ranks, [2.0, 0.5, 1.25], seed=560 + p)
            for p, (K, ranks) in enumerate(((264, [8, 24, 40]), (64, [16, 16, 33]), (72, [1, 32, 7])))]
    tens = [l.tensors() for l in lins]
    for t in tens[1:]:
        t.x = tens[0].x
    dps = [gh.upload(l, t, p % 2) for p, (l, t) in enumerate(zip(lins, tens))]
    group = plora.Group([dp.desc for dp in dps])
    guards: list = []
    ws = gh.guarded((plora.plora_group_workspace_bytes(group),), torch.uint8, None, guards, "group workspace")
    x = dps[0].x
    lists = lambda name: [getattr(dp, name) for dp in dps]

    def step():
        plora.plora_group_fwd(group, x, lists("W"), lists("A"), lists("B"), lists("y"), lists("h"), ws)
        plora.plora_group_bwd(group, x, lists("W"), lists("A"), lists("B"), lists("dy"), None, lists("dx"), lists("dA"), lists("dB"), ws)

    outputs = lambda: [b for dp in dps for b in (dp.y, dp.dx, dp.h, *dp.dA, *dp.dB)]

    def snapshot():
        torch.cuda.synchronize()
        return [b.clone() for b in outputs()]

    step()
    want = snapshot()
    say("[case] graph capture grouped")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        step()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=side):
            step()
    torch.cuda.synchronize()
    for rep in range(3):
        for buf in outputs():
            buf.fill_(float("nan"))
        ws.fill_(0xAB)
        torch.cuda.synchronize()
        graph.replay()
        got = snapshot()
        for a, b in zip(got, want):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), f"replay {rep} differs from the eager run"
    for dp in dps:
        gh.check_guards(dp)
    for name, base, nbytes in guards:
        assert bool((base[:gh.GUARD_BYTES] == gh.GUARD_BYTE).all()) and bool((base[gh.GUARD_BYTES + nbytes:] == gh.GUARD_BYTE).all()), name


@pytest.mark.parametrize("mode", ["saved", "recomputed", "lora_only", "noalloc", "grouped"])
def test_replay_of_short_products_with_several_shares(mode):
    """The workgroups of a short product that share a contraction announce themselves with a number that a captured launch keeps:
    every replay finds its flags at zero again, and sums what this replay wrote.  The inputs change between the replays, the
    workspace is left as the replay before left it, then scribbled over."""
    import torch
    import gpu_harness as gh
    Ks = (2504, 1032) if mode == "grouped" else (2504,)
    lora = mode == "lora_only"
    lins = [wl.small(f"graph_shares_{K}", "bf16", 1000, K, lengths=[300, 201], seg_adapter=[0, 1], ranks=[100, 7], scales=[2.0, 0.5],
                     seed=571 + p) for p, K in enumerate(Ks)]
    dps = [gh.upload(lin, lin.tensors(), lora_only=lora) for lin in lins]
    infos = [plora.plora_debug_metadata(dp.desc)[0] for dp in dps]
    assert all(min(i.short_shares) > 1 for i in infos)
    dp, x = dps[0], dps[0].x
    group = plora.Group([d.desc for d in dps])
    size = {"grouped": lambda: plora.plora_group_workspace_bytes(group), "lora_only": lambda: plora.plora_lora_workspace_bytes(dp.desc)}.get(
        mode, lambda: plora.plora_workspace_bytes(dp.desc))()
    ws, other_ws = torch.zeros(size, dtype=torch.uint8, device="cuda"), torch.zeros(size, dtype=torch.uint8, device="cuda")
    bases = [torch.randn_like(dp.y), torch.randn_like(dp.dx)]
    lists = lambda name: [getattr(d, name) for d in dps]

    def step(w, captured):
        h = None if mode == "recomputed" else dp.h
        if mode == "grouped":
            plora.plora_group_fwd(group, x, lists("W"), lists("A"), lists("B"), lists("y"), lists("h"), w)
            plora.plora_group_bwd(group, x, lists("W"), lists("A"), lists("B"), lists("dy"), None, lists("dx"), lists("dA"), lists("dB"), w)
        elif lora:
            dp.y.copy_(bases[0])
            dp.dx.copy_(bases[1])
            plora.plora_lora_fwd(dp.desc, x, dp.A, dp.B, dp.y, h, w)
            plora.plora_lora_bwd(dp.desc, x, dp.A, dp.B, dp.dy, h, dp.dx, dp.dA, dp.dB, w)
        elif mode == "noalloc" and captured:
            plora.plora_linear_fwd_noalloc(dp.desc, x, dp.W, dp.A, dp.B, dp.y, h)
        else:
            plora.plora_linear_fwd(dp.desc, x, dp.W, dp.A, dp.B, dp.y, h, w)
            if mode != "noalloc":
                plora.plora_linear_bwd(dp.desc, x, dp.W, dp.A, dp.B, dp.dy, h, dp.dx, dp.dA, dp.dB, w)

    backward = [] if mode == "noalloc" else [b for d in dps for b in (d.dx, *d.dA, *d.dB)]
    outputs = [b for d in dps for b in (d.y, d.h)] + backward

    def snapshot():
        torch.cuda.synchronize()
        return [b.clone() for b in outputs]

    inputs = [x] + lists("dy")
    sets = [[b.clone() for b in inputs], [torch.randn_like(b) for b in inputs], [torch.randn_like(b) for b in inputs]]

    def load(i):
        for b, v in zip(inputs, sets[i]):
            b.copy_(v)

    want = []
    for i in range(3):
        load(i)
        step(other_ws, False)
        want.append(snapshot())
    say(f"[case] graph, several shares, {mode}")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        step(ws, True)
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=side):
            step(ws, True)
    torch.cuda.synchronize()
    flags = []
    if mode not in ("noalloc", "lora_only"):                     # (their workspaces are laid out elsewhere)
        at = 0
        for d, i in zip(dps, infos):
            flags.append(ws[at + i.ws_flags:at + i.ws_flags + i.flag_bytes])
            at += (plora.plora_workspace_bytes(d.desc) + 255) // 256 * 256
    for rep in range(7):
        i = (0, 1, 2, 0, 1, 0, 2)[rep]
        load(i)
        for b in outputs:
            b.fill_(float("nan"))
        if rep >= 5:
            ws.fill_(0xAB)
        torch.cuda.synchronize()
        graph.replay()
        for a, b in zip(snapshot(), want[i]):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), f"replay {rep} differs from the eager run"
        assert rep >= 5 or all(f.numel() > 0 and not bool(f.any()) for f in flags), f"flags left behind by replay {rep}"
    for d in dps:
        gh.check_guards(d)
