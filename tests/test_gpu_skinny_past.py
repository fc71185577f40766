"""Shrink and dH of a matrix that is read past the caches (in a stand-alone call from 48 MB on, where its rows are whole lines of 128
bytes), of small ranks with every workgroup begun at another stage, against fp32 products of the same call; more than 64 token
blocks, ragged rows, a shorter last split."""
import numpy as np
import pytest

from paper_2508_02932_amd import plora

pytestmark = pytest.mark.gpu
TOL = 2e-2


@pytest.mark.parametrize("ranks", [(16, 9, 32), (48, 128, 3)], ids=["turned", "wide"])
@pytest.mark.parametrize("D,K", [(72, 8256), (8256, 72), (72, 8264), (8264, 72)])
def test_large_matrix(D, K, ranks):
    import torch
    lengths = [1 + 37 * i % 97 for i in range(66)]
    T = sum(lengths)
    assert T * 8256 * 2 >= 48 << 20
    off, owner = np.concatenate([[0], np.cumsum(lengths)]), np.array([i % 3 for i in range(66)])
    scales = [2.0, 0.5, 1.25]
    d = plora.Desc(T, D, K, off, owner, np.array(ranks), np.array(scales), plora.PLORA_BF16)
    info = plora.plora_debug_metadata(d)[0]
    assert info.short_shares[0 if D > K else 1] == 0 and max(info.shrink_splits, info.dh_splits) > 1
    print(f"[case] {D} -> {K} ranks {ranks}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(487)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g).to(torch.bfloat16)
    x, dy, y0, dx0 = rnd(T, D), rnd(T, K), rnd(T, K), rnd(T, D)
    A, B = [rnd(D, r) for r in ranks], [rnd(r, K) for r in ranks]
    y, dx = y0.clone(), dx0.clone()
    dA, dB = [torch.empty(D, r, device="cuda") for r in ranks], [torch.empty(r, K, device="cuda") for r in ranks]
    h = torch.empty(plora.plora_h_elems(d), dtype=torch.float32, device="cuda")
    ws = torch.empty(plora.plora_lora_workspace_bytes(d), dtype=torch.uint8, device="cuda")
    plora.plora_lora_fwd(d, x, A, B, y, h, ws)
    plora.plora_lora_bwd(d, x, A, B, dy, h, dx, dA, dB, ws)
    torch.cuda.synchronize()
    want_y, want_dx = y0.float(), dx0.float()
    want_dA, want_dB = [torch.zeros_like(t) for t in dA], [torch.zeros_like(t) for t in dB]
    at, errs = 0, {}
    err = lambda got, want: float((got.float() - want).abs().max() / want.abs().max())
    for s, k in enumerate(owner):
        lo, hi, r = int(off[s]), int(off[s + 1]), ranks[k]
        hs = x[lo:hi].float() @ A[k].float()
        gs = scales[k] * (dy[lo:hi].float() @ B[k].float().t())
        errs["h"] = max(errs.get("h", 0.0), err(h[at:at + (hi - lo) * r].view(hi - lo, r), hs))
        at += (hi - lo) * r
        want_y[lo:hi] += scales[k] * (hs @ B[k].float())
        want_dx[lo:hi] += gs @ A[k].float().t()
        want_dA[k] += x[lo:hi].float().t() @ gs
        want_dB[k] += scales[k] * (hs.t() @ dy[lo:hi].float())
    errs.update(y=err(y, want_y), dx=err(dx, want_dx))
    for k in range(3):
        errs[f"dA{k}"], errs[f"dB{k}"] = err(dA[k], want_dA[k]), err(dB[k], want_dB[k])
    print("  errors " + " ".join(f"{n}={v:.2e}" for n, v in errs.items()), flush=True)
    assert all(np.isfinite(v) and v <= TOL for v in errs.values()), errs
