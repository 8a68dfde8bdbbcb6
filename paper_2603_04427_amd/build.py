"""Builds libtkattn.so (the HIP kernels and the C ABI) for gfx950 with hipcc,
beside it _tkcall.so, the call path from torch tensors to the C ABI (host code,
against the installed torch), and libtkprobe.so, the benchmark's streaming-read
probe.

Usage: python -m paper_2603_04427_amd.build   (or build() from Python).
Objects go to _build/ at the repository root; the library lands next to this
file so that it travels with the package.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libtkattn.so")
PROBE_LIB = os.path.join(PKG, "libtkprobe.so")
PROBE_SOURCE = "stream_probe.hip"
CALL_LIB = os.path.join(PKG, "_tkcall.so")
CALL_SOURCE = "torch_call.cpp"
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SOURCES = ["api.cpp", "decode.hip", "decode_short.hip", "prefill_bf16.hip", "prefill_f32.hip", "prefill_bwd.hip", "append.hip", "project.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-I" + INCLUDE, "-I" + CSRC,
         # packed fp32 arithmetic stays off: ordinary fp32 code only
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         # matrix-core accumulators in ordinary VGPRs: the softmax reads the score
         # tiles directly and the output tiles do not bounce through AGPRs
         "-mllvm", "-amdgpu-mfma-vgpr-form=1",
         "-Wall", "-Wno-unused-result"]


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC] + FLAGS + ["-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    return obj


def _link(objs, lib: str) -> None:
    tmp = lib + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, lib)


def _build_call_path() -> None:
    import sysconfig

    import torch
    from torch.utils import cpp_extension

    libs = os.path.join(os.path.dirname(torch.__file__), "lib")
    rocm = os.path.dirname(os.path.dirname(HIPCC))
    includes = [INCLUDE, sysconfig.get_paths()["include"], os.path.join(rocm, "include")] + cpp_extension.include_paths()
    tmp = CALL_LIB + ".tmp"
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"]
    cmd += ["-isystem" + d if d != INCLUDE else "-I" + d for d in includes]
    cmd += [os.path.join(CSRC, CALL_SOURCE), "-o", tmp, "-L" + libs, "-Wl,-rpath," + libs,
            "-ltorch_python", "-ltorch_cpu", "-ltorch", "-lc10_hip", "-lc10"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"g++ failed for {CALL_SOURCE}:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, CALL_LIB)


def build(verbose: bool = False) -> str:
    """Compile every source and link the shared libraries. Returns libtkattn's path."""
    os.makedirs(BUILD, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=min(len(SOURCES) + 2, os.cpu_count() or 4)) as ex:
        call_path = ex.submit(_build_call_path)
        objs = list(ex.map(_compile, SOURCES + [PROBE_SOURCE]))
        call_path.result()
    _link(objs[:-1], LIB)
    _link(objs[-1:], PROBE_LIB)
    if verbose:
        print(f"built {LIB}, {CALL_LIB} and {PROBE_LIB}")
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
