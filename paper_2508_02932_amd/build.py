"""Builds libplora.so (HIP kernels + C ABI) for gfx950 with hipcc, and the binding's marshalling module, in-tree."""
from __future__ import annotations

import os
import re
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libplora.so")
BENCH_LIB = os.path.join(HERE, "libplora_bench.so")      # ceiling microkernels for bench.py, not the product
BINDING = os.path.join(HERE, "_plora_binding.so")         # marshalling for plora.py
SOURCES = ["plora_api.hip", "small_kernels.hip", "f32_kernels.hip", "skinny_bf16.hip",
           "gemm_bf16.hip", "gemm_small_bf16.hip", "gemm_short_bf16.hip", "tokcontract_bf16.hip", "adamw.hip", "expand_bf16.hip", "nf4.hip",
           "planner.cpp"]                                     # host only: the packing planner
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC]

# Sources with kernels on the fp64 matrix instruction (f32_tiles.h): their sums must lie in ordinary vector registers.
F64_SOURCES = ("f32_kernels.hip", "small_kernels.hip")
REMARK = "kernel-resource-usage"


def kernels_with_accumulation_registers(remarks: str) -> list:
    """The fp32 path's kernels (k_f32_*, k_prep_f32) that the compiler's resource remarks give accumulation registers."""
    found, name = [], ""
    seen = 0
    for line in remarks.splitlines():
        m = re.search(r"remark: Function Name: (\S+)", line)
        if m:
            name = m.group(1)
        m = re.search(r"remark:\s+AGPRs: (\d+)", line)
        if m and re.search(r"k_f32_|k_prep_f32", name):
            seen += 1
            if int(m.group(1)) > 0:
                found.append(name)
    if not seen:
        raise RuntimeError("no resource remarks of the fp32 path's kernels")
    return found


def _compile(src: str, obj_dir: str = OBJ, extra=()) -> str:
    obj = os.path.join(obj_dir, os.path.splitext(src)[0] + ".o")
    checked = src in F64_SOURCES
    flags = ["-Rpass-analysis=" + REMARK, "-fno-caret-diagnostics"] if checked else []
    cmd = ["hipcc", *FLAGS, *flags, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    lines = res.stderr.splitlines()
    err = "\n".join(l for l in lines if "packed-fp32-ops" not in l and "argument unused during compilation" not in l and REMARK not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if checked:
        bad = kernels_with_accumulation_registers("\n".join(l for l in lines if REMARK in l))
        if bad:
            raise RuntimeError(f"{src}: sums in accumulation registers, which are read too early (see f32_tiles.h): {', '.join(bad)}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build_binding() -> str:
    """The marshalling module of plora.py (host code against the headers of the installed torch)."""
    import torch
    inc = os.path.join(torch.__path__[0], "include")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-I", os.path.join(ROOT, "include"), "-isystem", inc, "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"),
           "-isystem", sysconfig.get_paths()["include"], os.path.join(CSRC, "binding.cpp"), "-o", BINDING,
           "-L", os.path.join(torch.__path__[0], "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("g++ failed on binding.cpp:\n" + res.stderr)
    if res.stderr.strip():
        sys.stderr.write(res.stderr + "\n")
    return BINDING


def build(verbose: bool = False) -> str:
    """Compile every HIP source and link the shared library.  Always recompiles."""
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=8) as ex:
        binding = ex.submit(build_binding)
        objs = list(ex.map(_compile, SOURCES + ["bench_ceilings.hip"]))
        binding.result()
    if verbose:
        print("built", BINDING)
    for lib, parts in ((LIB, objs[:-1]), (BENCH_LIB, objs[-1:])):
        cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", lib, *parts]
        res = subprocess.run(cmd, capture_output=True, text=True)
        if res.returncode != 0:
            raise RuntimeError("link failed:\n" + res.stderr)
        if verbose:
            print("built", lib)
    return LIB


def build_variant(lib_path: str, extra_flags, sources=("gemm_bf16.hip",)) -> str:
    """A copy of libplora.so at lib_path in which `sources` are compiled with extra flags (tuning runs; the other
    objects are taken from the last regular build)."""
    obj_dir = lib_path + ".obj"
    os.makedirs(obj_dir, exist_ok=True)
    objs = []
    for src in SOURCES:
        if src in sources:
            objs.append(_compile(src, obj_dir, tuple(extra_flags)))
        else:
            objs.append(os.path.join(OBJ, os.path.splitext(src)[0] + ".o"))
    res = subprocess.run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", lib_path, *objs], capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("link failed:\n" + res.stderr)
    return lib_path


if __name__ == "__main__":
    build(verbose=True)
