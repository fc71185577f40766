"""The work that bench.py divides a kernel class's time by, and the line that bench.py prints: one JSON object with the required keys, short enough that a log which keeps the last 2000
characters of a run keeps all of it, whatever else was measured."""
import json

import bench

REQUIRED = ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline", "dtype",
            "data", "config")


def full_record():
    entry = {"ms": 12.3456, "bound": "mfma", "achieved": 1234.5, "unit": "TFLOP/s", "frac": 0.1234, "algorithmic_bytes": 2012989536,
             "frac_of_measured_ceiling": 0.1234, "note": "n" * 120}
    names = ("gemm_fwd", "gemm_dx", "shrink", "dh", "db", "da", "adamw")
    kernels = dict({n: entry for n in names}, prep={"ms": 0.0229})
    return {"metric": "packed multi-LoRA layer fwd+bwd TFLOP/s", "value": 1234.56, "unit": "TFLOP/s", "tokens_per_s": 12345678.9, "n_gpus": 1,
            "steps": 1000, "warmup": 100, "ms_per_step": 12.3456, "step_ms": {"median_ms": 12.3456, "min_ms": 12.3456, "max_ms": 12.3456},
            "host_us_per_call": {"fwd": 12.3, "bwd": 12.3}, "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "bf16",
            "data": "synthetic",
            "config": {"workload": "config 5 / c5_mlp_up: d_in=8192 d_out=28672 T=32768 adapters=32 ranks=" + str(list(range(8, 129, 8)))
                                   + " W stored [d_out][d_in]", "tokens": 32768, "d_in": 8192, "d_out": 28672, "n_adapters": 32,
                       "flops_per_step": 31042161803264.0},
            "frac_of_bf16_mfma_peak": 0.1234,
            "roofline": {"kernel": "k_gemm<forward> (x W with fused scale*h*B_k)", "bound": "mfma", "achieved": 1234.5, "peak": 2500.0,
                         "unit": "TFLOP/s", "frac": 0.1234, "traffic": 28300000000.0, "avg_launch_ms": 12.3456,
                         "frac_of_measured_ceiling": 0.1234},
            "kernels": kernels, "measured_ceilings": {"stream_read_gbs": 5700.0},
            "per_config": [{"workload": "w" * 60, "kernels": kernels}] * 20, "planner": {"note": "n" * 900},
            "cpu_baseline": {"value": 0.091234, "unit": "TFLOP/s", "cores": 16, "kind": "oracle", "tokens_per_s": 1234.56,
                             "sample": "fp64 scalar-loop oracle: y and dx of 32768 random rows of 32768 (10.0 s) plus dA, dB of 32 of 32 adapters "
                                       "(10.0 s); whole step extrapolated: row part scaled by T / rows, weight gradients by sum(L r)"}}


def test_the_printed_line_is_whole_in_a_short_log():
    line = json.dumps(bench.printed_line(full_record(), "/tmp/plora_bench_record.json"))
    assert len(line) <= bench.LINE_CHARS < 2000
    got = json.loads(line)
    assert all(k in got for k in REQUIRED) and got["roofline"]["frac"] == 0.1234 and got["cpu_baseline"]["value"] == 0.091234
    assert got["kernels"]["gemm_fwd"] == {"ms": 12.3456, "frac": 0.1234} and got["kernels"]["prep"] == {"ms": 0.0229}
    long = full_record()
    long["config"]["workload"] += " " * 400
    got = json.loads(json.dumps(bench.printed_line(long, "/tmp/plora_bench_record.json")))
    assert len(json.dumps(got)) <= bench.LINE_CHARS and all(k in got for k in REQUIRED) and "kernels" not in got


def test_work_of_the_fp32_weight_gradients_is_that_of_their_one_launch():
    from paper_2508_02932_amd import workloads as wl
    f, b = (wl.small("work", t, 64, 48, lengths=[30, 20], seg_adapter=[0, 1], ranks=[8, 4], scales=[1.0, 1.0], seed=1) for t in ("f32", "bf16"))
    T, D, K, R, Lr = 50, 64, 48, 12, 30 * 8 + 20 * 4
    assert "da" not in bench.work_of(f)
    assert bench.work_of(f)["db"] == ("hbm", T * (D + K) * 4 + 2 * Lr * 4 + R * (D + K) * 4)
    assert bench.work_of(b)["db"] == ("hbm", T * K * 2 + Lr * 4 + R * K * 4) and bench.work_of(b)["da"] == ("hbm", T * D * 2 + Lr * 4 + D * R * 4)


def test_main_shadows_no_function_of_the_module():
    functions = {n for n, v in vars(bench).items() if callable(v) and getattr(v, "__module__", None) == "bench"}
    assert not functions & set(bench.main.__code__.co_varnames + bench.main.__code__.co_cellvars)
