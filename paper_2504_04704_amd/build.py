"""Builds liblagkv.so (the C-ABI library) in-tree with hipcc for gfx950."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG_DIR)
CSRC = os.path.join(PKG_DIR, "csrc")
LIB_PATH = os.path.join(PKG_DIR, "liblagkv.so")
BINDING_PATH = os.path.join(PKG_DIR, "_lagkv_native.so")
SOURCES = ["lagkv_api.hip", "split_pass.hip", "hold_pass.hip", "append_pass.hip", "staged_pass.hip",
           "chunk_f32.hip", "chunk_bf16.hip", "chunk_f16.hip",
           "ring_f32.hip", "ring_bf16.hip", "ring_f16.hip",
           "round_f32.hip", "round_bf16.hip", "round_f16.hip", "static_scratch.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed fp32 VALU ops are kept off on this target
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def hipcc_path() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def _run(cmd, verbose):
    if verbose:
        print("[build]", " ".join(cmd), flush=True)
    proc = subprocess.run(cmd, capture_output=True, text=True)
    out = (proc.stdout + proc.stderr).strip()
    # the host pass does not know the gfx feature name; that warning is harmless
    out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
    if verbose and out:
        print(out, flush=True)
    if proc.returncode != 0:
        raise RuntimeError(f"{os.path.basename(cmd[0])} failed ({proc.returncode})\n{out}")


def build_library(verbose: bool = True, extra_flags=(), out_path: str = LIB_PATH, sources=SOURCES) -> str:
    """Compile every HIP source (one hipcc process per file) and link them into
    paper_2504_04704_amd/liblagkv.so; returns its path."""
    hipcc = hipcc_path()
    inc = ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
    with tempfile.TemporaryDirectory(prefix="lagkv_build_") as tmp:
        objs = [os.path.join(tmp, os.path.splitext(s)[0] + ".o") for s in sources]
        cmds = [[hipcc, *HIPCC_FLAGS, *extra_flags, *inc, "-c", os.path.join(CSRC, s), "-o", o]
                for s, o in zip(sources, objs)]
        with ThreadPoolExecutor(min(len(cmds), os.cpu_count() or 1, 8)) as ex:
            list(ex.map(lambda c: _run(c, verbose), cmds))
        _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", out_path + ".tmp"], verbose)
    os.replace(out_path + ".tmp", out_path)
    return out_path


def build_binding(verbose: bool = True, out_path: str = BINDING_PATH) -> str:
    """Compile csrc/binding.cpp (host code only, against torch's headers) into paper_2504_04704_amd/_lagkv_native.so, with
    g++ or, where there is none, the clang that hipcc drives; returns its path."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension
    cxx = [shutil.which("g++") or shutil.which("c++")]
    if cxx[0] is None:
        cxx = [hipcc_path(), "-x", "c++"]
    inc = [*cpp_extension.include_paths(), sysconfig.get_paths()["include"], os.path.join(ROOT, "include"), CSRC]
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    _run([*cxx, "-O2", "-std=c++17", "-shared", "-fPIC", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
          *(x for i in inc for x in ("-isystem", i)), os.path.join(CSRC, "binding.cpp"), "-o", out_path + ".tmp",
          "-L", lib, "-lc10", "-ltorch_cpu", "-ltorch_python", f"-Wl,-rpath,{lib}"], verbose)
    os.replace(out_path + ".tmp", out_path)
    return out_path


if __name__ == "__main__":
    build_library(extra_flags=sys.argv[1:])
    build_binding()
