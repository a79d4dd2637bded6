"""Build the HIP C-ABI library (liblemo_hip.so) for gfx950 with hipcc, in-tree.

Usage: ``python -m paper_2501_09767_amd.build`` or ``build_library()``.  Cross-compiles without a GPU.
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJDIR = os.path.join(ROOT, "_build")
LIB = os.path.join(HERE, "liblemo_hip.so")
NATIVE = os.path.join(HERE, "lemo_native.so")  # the binding's native marshalling, linked against LIB
SOURCES = ["lemo_api.hip", "score.hip", "score_f32.hip", "score_blocks.hip", "score_blocks_few.hip", "score_blocks_slabs.hip", "attention.hip", "select.hip", "gather_gemm.hip", "gather_gemm_large.hip", "gather_gemm_mid.hip", "gather_gemm_small.hip", "transpose.hip", "scatter.hip", "probe.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# packed-fp32 code generation is switched off on purpose: the compiler must not form v_pk_*_f32 instructions from scalar float code
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-command-line-argument",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]


# Per-file flags.  attention.hip (its 64-queries-per-wave kernel) and score_blocks_few.hip may use the whole register file
# (one wave per SIMD), and for such a kernel the compiler would otherwise give every MFMA its result in the accumulation
# registers, with a copy around each use by vector arithmetic; this makes MFMAs write ordinary vector registers.
FILE_FLAGS = {"attention.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"], "score_blocks_few.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"]}


def _compile(src: str, extra) -> str:
    obj = os.path.join(OBJDIR, src.replace(".hip", ".o"))
    cmd = [HIPCC, *FLAGS, *FILE_FLAGS.get(src, []), *extra, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        print(err, file=sys.stderr)
    return obj


def build_native() -> str:
    """csrc/native.cpp as a CPython extension beside the library (host compiler, torch's headers)."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension

    tmp = NATIVE + f".tmp{os.getpid()}"
    libs = cpp_extension.library_paths()
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}",
           f'-DLEMO_TORCH_VERSION="{torch.__version__}"',
           "-I" + os.path.join(ROOT, "include"), "-I" + sysconfig.get_paths()["include"], *("-isystem" + p for p in cpp_extension.include_paths()),
           os.path.join(CSRC, "native.cpp"), "-o", tmp, "-L" + HERE, "-l:liblemo_hip.so", "-Wl,-rpath,$ORIGIN",
           *("-L" + p for p in libs), *("-Wl,-rpath," + p for p in libs), "-lc10", "-ltorch_cpu", "-ltorch_python"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("building the native binding failed:\n" + r.stderr)
    if r.stderr.strip():
        print(r.stderr, file=sys.stderr)
    os.replace(tmp, NATIVE)
    return NATIVE


def build_library(extra_flags=(), verbose: bool = True) -> str:
    os.makedirs(OBJDIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(lambda s: _compile(s, list(extra_flags)), SOURCES))
    tmp = LIB + f".tmp{os.getpid()}"
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs], capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    os.replace(tmp, LIB)
    native = build_native()
    if verbose:
        print("built", LIB, native)
    return LIB


if __name__ == "__main__":
    build_library(sys.argv[1:])
