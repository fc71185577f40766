"""The stand-alone low-rank update of an output larger than the last cache (256 MB), which is read and written past it, against the
same rows in two calls below that size: the same operations on every element, so the same bits.  Ragged rows and column tiles, one
case for each number of rank steps that the kernel is built for, and one whose rows are not whole lines of 128 bytes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rank,K", [(16, 64064), (63, 64064), (128, 64064), (16, 64008)])
def test_large_output_is_bitwise_its_halves(rank, K):
    import torch
    from paper_2508_02932_amd import plora
    cuts, D = [0, 1, 530, 1050, 1051, 1700, 2100], 64
    assert 2100 * K * 2 > 256 << 20 > 1050 * K * 2
    print(f"[case] lora-only 2100 x {K} rank {rank}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(461)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g).to(torch.bfloat16)
    x, A, B, y0 = rnd(2100, D), rnd(D, rank), rnd(rank, K), rnd(2100, K)

    def update(lo, hi):
        off = np.array([c - cuts[lo] for c in cuts[lo:hi + 1]])
        d = plora.Desc(int(off[-1]), D, K, off, np.zeros(hi - lo), np.array([rank]), np.array([0.5]), plora.PLORA_BF16)
        ws = torch.empty(plora.plora_lora_workspace_bytes(d), dtype=torch.uint8, device="cuda")
        y = y0[cuts[lo]:cuts[hi]].clone()
        plora.plora_lora_fwd(d, x[cuts[lo]:cuts[hi]].clone(), [A], [B], y, None, ws)
        torch.cuda.synchronize()
        return y

    whole, first, second = update(0, 6), update(0, 3), update(3, 6)
    assert torch.equal(whole[:1050], first) and torch.equal(whole[1050:], second)
    want = y0[:64].float() + 0.5 * ((x[:64].float() @ A.float()).to(torch.bfloat16).float() @ B.float())
    assert float((whole[:64].float() - want).abs().max()) <= 2e-2 * float(want.abs().max())
