"""The launches of the device entry points, on the CPU: a recorder in place of the HIP runtime takes them down and runs nothing.
A kernel that is given more than the 64 KB of dynamic LDS that every kernel may have must have been allowed them first."""
import json
import os
import random
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DEFAULT_LDS = 64 << 10


def calls_driver(jobs):
    """Runs in a process of its own with the recorder preloaded: [(operation, [description of every projection])] -> launches."""
    import ctypes as C
    import numpy as np
    from paper_2508_02932_amd import plora
    L, rec = plora.lib(), C.CDLL(os.environ["PLORA_RECORDER"])
    rec.recorder_kernel.restype = C.c_char_p
    for f in (rec.recorder_workgroups, rec.recorder_lds, rec.recorder_allowed):
        f.restype = C.c_uint64
    keep, at = [], [1 << 40]

    def address(n_bytes):                             # of device memory that nobody reads
        at[0] += (n_bytes + (1 << 20)) // 256 * 256
        return at[0]

    def table(addresses):
        keep.append((C.c_void_p * max(1, len(addresses)))(*addresses))
        return C.addressof(keep[-1])

    out = []
    for op, projections in jobs:
        descs = [plora.Desc(sum(lengths), D, K, np.concatenate([[0], np.cumsum(lengths)]), np.array(owner), np.array(ranks), np.ones(len(ranks)), dtype, w)
                 for D, K, lengths, owner, ranks, dtype, w in projections]
        d = descs[0]
        e = 2 if d.dtype == plora.PLORA_BF16 else 4
        x = address(d.T * d.d_in * e)
        side = lambda width, size: [table([address(size * int(r) * width(q)) for r in q.rank]) for q in descs]
        A, B = side(lambda q: q.d_in, e), side(lambda q: q.d_out, e)
        dA, dB = side(lambda q: q.d_in, 4), side(lambda q: q.d_out, 4)
        one = lambda size: [address(size(q)) for q in descs]
        W, y, dy = one(lambda q: q.d_in * q.d_out * e), one(lambda q: q.T * q.d_out * e), one(lambda q: q.T * q.d_out * e)
        h, dx = one(lambda q: 4 * plora.plora_h_elems(q)), one(lambda q: q.T * q.d_in * e)
        size = {"lora": L.plora_lora_workspace_bytes, "nf4": L.plora_nf4_workspace_bytes}.get(op, L.plora_workspace_bytes)(d.ref)
        ws, absmax = address(size), address(d.d_in * d.d_out // 16)
        rec.recorder_clear()
        if op == "noalloc":
            codes = [L.plora_linear_fwd_noalloc(d.ref, x, W[0], A[0], B[0], y[0], h[0], None)]
        elif op == "step":
            codes = [L.plora_linear_fwd(d.ref, x, W[0], A[0], B[0], y[0], h[0], ws, size, None)]
            for saved in (h[0], None):
                codes.append(L.plora_linear_bwd(d.ref, x, W[0], A[0], B[0], dy[0], saved, dx[0], dA[0], dB[0], ws, size, None))
            codes.append(L.plora_linear_bwd(d.ref, x, W[0], A[0], B[0], dy[0], h[0], dx[0], None, None, ws, size, None))
        elif op == "lora":
            codes = [L.plora_lora_fwd(d.ref, x, A[0], B[0], y[0], h[0], ws, size, None),
                     L.plora_lora_bwd(d.ref, x, A[0], B[0], dy[0], h[0], dx[0], dA[0], dB[0], ws, size, None)]
        elif op == "nf4":
            codes = [L.plora_linear_fwd_nf4(d.ref, x, W[0], absmax, A[0], B[0], y[0], None, ws, size, None),
                     L.plora_linear_bwd_nf4(d.ref, x, W[0], absmax, A[0], B[0], dy[0], None, dx[0], dA[0], dB[0], ws, size, None)]
        else:
            group = plora.Group(descs)
            size = L.plora_group_workspace_bytes(C.byref(group.c))
            ws = address(size)
            codes = [L.plora_group_fwd(C.byref(group.c), x, table(W), table(A), table(B), table(y), table(h), ws, size, None),
                     L.plora_group_bwd(C.byref(group.c), x, table(W), table(A), table(B), table(dy), table(h), None, dx[0], table(dA), table(dB), ws, size, None)]
        out.append((codes, [(rec.recorder_kernel(i).decode(), rec.recorder_workgroups(i), rec.recorder_lds(i), rec.recorder_allowed(i))
                            for i in range(rec.recorder_count())]))
    return out


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("recorder") / "librecorder.so")
    res = subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", lib, os.path.join(ROOT, "tests", "launch_recorder.cpp")],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]

    def record(jobs):
        """Of every job: the kernels' names with workgroups, dynamic LDS and how much of that was allowed.  A process per call of this:
        what a kernel is allowed lasts as long as the process."""
        code = "import json, sys; sys.path[:0] = [%r, %r]; import test_launches_host as t; print(json.dumps(t.calls_driver(json.load(sys.stdin))))" % (
            ROOT, os.path.join(ROOT, "tests"))
        run = subprocess.run([sys.executable, "-c", code], input=json.dumps(jobs), capture_output=True, text=True, timeout=600,
                             env=dict(os.environ, PLORA_RECORDER=lib, LD_PRELOAD=":".join([lib] + [v for v in [os.environ.get("LD_PRELOAD")] if v])))
        assert run.returncode == 0, run.stderr[-3000:]
        out = json.loads(run.stdout)
        assert len(out) == len(jobs) and all(code == 0 for codes, _ in out for code in codes)
        return [calls for _, calls in out]
    return record


def refused(calls):
    return [(kernel, lds) for kernel, _, lds, allowed in calls if lds > max(allowed, DEFAULT_LDS)]


# d_in, d_out, lengths, owners, ranks: the finishing launch of a forward in two launches with four blocks of columns and four steps of rank
WIDE = {
    "unsplit": (1496, 5680, [120, 130, 129], [0, 1, 2], [8, 117, 30]),
    "split": (4096, 7168, [200, 100], [0, 1], [112, 16]),
    "ragged": (2048, 4200, [90, 310, 100], [0, -1, 1], [16, 128]),
}


@pytest.mark.parametrize("projections", [1, 2])
@pytest.mark.parametrize("w", [0, 1])
@pytest.mark.parametrize("case", sorted(WIDE))
def test_wide_finish_is_allowed_its_lds(launches, case, w, projections):
    shape = (*WIDE[case], 0, w)
    (calls,) = launches([("noalloc", [shape]) if projections == 1 else ("group", [shape] * projections)])
    (lds,) = [lds for kernel, _, lds, _ in calls if "k_short_finish" in kernel]
    assert lds > DEFAULT_LDS
    assert refused(calls) == []


def random_jobs(seed, n):
    rng = random.Random(seed)
    jobs = []
    for _ in range(n):
        op = rng.choice(["noalloc", "step", "step", "lora", "nf4", "group"])
        n_ad = rng.choice([1, 2, 5, 8, 20])
        parts = rng.choice([1, n_ad, n_ad + 3])
        T = int(2 ** rng.uniform(3, 13))
        lengths = [T // parts + (i < T % parts) for i in range(parts)]
        ranks = [rng.choice([1, 8, 16, 33, 64, 100, 128]) for _ in range(n_ad)]
        D, K = 64 * int(2 ** rng.uniform(1, 7)), 64 * int(2 ** rng.uniform(1, 7))
        if op == "noalloc":
            T = min(T, 512)
            lengths = [T // parts + (i < T % parts) for i in range(parts)]
        shape = lambda K: (D, K, lengths, [i % (n_ad + 1) - 1 if i >= n_ad else i for i in range(parts)], ranks, 1 if rng.random() < 0.1 and op != "group" else 0,
                           rng.randint(0, 1))
        jobs.append((op, [shape(K) for _ in range(rng.randint(1, 4) if op == "group" else 1)]))
    return jobs


def test_no_launch_takes_more_lds_than_it_was_allowed(launches):
    seen = set()
    for calls in launches(random_jobs(733, 60)):
        assert calls and refused(calls) == []
        seen.update(kernel for kernel, _, lds, _ in calls if lds > DEFAULT_LDS)
    for part in ("k_gemmI", "k_gemm_small", "k_tokcI", "k_short_products", "k_grads"):
        assert any(part in kernel for kernel in seen), part
