"""The records the skinny and weight-gradient kernels start from (one per token block, one per adapter) against the tables
they gather, as read back from the workspace: integers, compared exactly; and the finishing kernels at ranks and widths
around their tiles (16 rows, 64 columns) with a split token walk."""
import numpy as np
import pytest

import oracle
from paper_2508_02932_amd import workloads as wl
from test_gpu_parity import run_and_compare

pytestmark = pytest.mark.gpu

SEG = [("row0", "<i4"), ("row1", "<i4"), ("adapter", "<i4"), ("r", "<i4"), ("rp", "<i4"), ("r16", "<i4"), ("blk0", "<i4"), ("lp", "<i4"),
       ("h_off", "<i8"), ("hb_off", "<i8"), ("zt_off", "<i8")]
BLK = np.dtype(SEG + [("t0", "<i4"), ("scale", "<f4"), ("at_off", "<i8"), ("B", "<u8"), ("rp_off", "<i4"), ("reserved", "<i4")])
JOB = np.dtype([("dA", "<u8"), ("dB", "<u8"), ("zt_off", "<i8")] + [(n, "<i4") for n in ("row0", "len", "lp", "k", "r", "r16", "r16_off")]
               + [("scale", "<f4")] + [(n, "<i4") for n in ("seg_list0", "n_own", "n_steps", "reserved")])


def align(v):
    return (v + 63) // 64 * 64


def test_records_repeat_the_tables():
    import torch
    import gpu_harness as gh
    from paper_2508_02932_amd import plora
    lengths = [130, 0, 257, 64, 249, 1, 700, 30, 12] + [3] * 300
    owner = [1, 0, 2, -1, 1, 0, 3, 2, 0] + [i % 6 - 1 for i in range(300)]
    lin = wl.small("records", "bf16", 136, 264, lengths=lengths, seg_adapter=owner, ranks=[8, 24, 72, 128, 5, 9],
                   scales=[2.0, 0.5, 1.25, 1.0, 3.0, 4.0], seed=401)
    dp = gh.upload(lin, lin.tensors())
    gh.forward(dp)
    gh.backward(dp)
    torch.cuda.synchronize()
    info, _, _ = plora.plora_debug_metadata(dp.desc)
    dev = dp.ws[info.ws_meta:info.ws_meta + info.table_bytes].cpu().numpy()
    tab = plora.parse_tables(info, dev)
    at = align(int(info.off_tile_order) + 4 * int(info.n_tiles))
    blk = np.frombuffer(dev, BLK, info.n_blocks, at)
    job = np.frombuffer(dev, JOB, info.n_adapters, align(at + BLK.itemsize * info.n_blocks))
    for b, rec in enumerate(blk):
        s = int(tab["blk_seg"][b])
        for name, _ in SEG:
            assert rec[name] == tab["seg"][s][name], (b, name)
        a = tab["ad"][int(rec["adapter"])]
        assert rec["t0"] == 128 * (b - int(rec["blk0"]))
        assert (rec["scale"], rec["at_off"], rec["B"]) == (a["scale"], a["at_off"], a["B"])
        assert int(rec["rp_off"]) * 136 == int(a["ap_off"])                 # the padded operand has d_in rows here
    for i, rec in enumerate(job):
        k = int(rec["k"])
        assert k == int(tab["ad"][i]["by_tokens"])
        a = tab["ad"][k]
        for name in ("dA", "dB", "r", "r16", "r16_off", "scale", "seg_list0", "n_own"):
            assert rec[name] == a[name], (i, name)
        own = [int(tab["seg_list"][int(a["seg_list0"]) + j]) for j in range(int(a["n_own"]))]
        assert int(rec["n_steps"]) == sum(int(tab["seg"][s]["lp"]) // 64 for s in own)
        if own:
            g = tab["seg"][own[0]]
            assert (rec["row0"], rec["len"], rec["lp"], rec["zt_off"]) == (g["row0"], g["row1"] - g["row0"], g["lp"], g["zt_off"])


@pytest.mark.parametrize("D,K,ranks", [(72, 200, [1, 17]), (264, 56, [16, 33]), (328, 392, [128, 15])])
def test_split_token_walk(D, K, ranks):
    lin = wl.small(f"split_{D}_{K}", "bf16", D, K, lengths=[2100, 70, 1900, 33], seg_adapter=[0, 1, 1, 0], ranks=ranks,
                   scales=[2.0, 0.5], seed=409)
    from paper_2508_02932_amd import plora
    import gpu_harness as gh
    info, _, _ = plora.plora_debug_metadata(gh.desc_of(lin))
    assert info.da_splits > 1 and info.db_splits > 1
    run_and_compare(lin, impl=oracle.matmul)
