"""Build libtm_w4.so and the native half of the Python binding (tm_calls.so) in-tree with hipcc for gfx950
(cross-compiles without a GPU)."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libtm_w4.so")
CALLS = os.path.join(PKG, "tm_calls.so")
SOURCES = ["tm_w4_api.hip", "tm_w4_pack.hip", "tm_w4_skinny.hip", "tm_w4_stream.hip", "tm_w4_stream_grouped.hip", "tm_w4_streamx.hip", "tm_w4_streamx64.hip", "tm_w4_skinny_w8.hip", "tm_w4_skinny_f8.hip", "tm_w4_tile_small.hip", "tm_w4_tile_large.hip", "tm_w4_tile32.hip",
           "tm_w4_tile_kgroup.hip", "tm_w4_tile_grouped.hip", "tm_w4_tile_w8.hip", "tm_attn.hip", "tm_attn_prefill.hip"]
# per-file extra flags (see the header comment of each file)
EXTRA = {"tm_attn_prefill.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"],
         "tm_w4_tile_small.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"],
         "tm_w4_tile_kgroup.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"],
         "tm_w4_tile_grouped.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"],
         "tm_w4_tile_w8.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"]}
FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-fvisibility=hidden",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function", "-Wno-unused-command-line-argument"]


def build(verbose: bool = False, jobs: int = 8) -> str:
    """Compile every translation unit and link the two shared objects.  Always rebuilds."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    out = LIB
    objdir = os.path.join(PKG, "_build")
    os.makedirs(objdir, exist_ok=True)
    procs = []
    objs = []
    for src in SOURCES:
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        objs.append(obj)
        cmd = [hipcc, *FLAGS, *EXTRA.get(src, []), "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        if len(procs) >= jobs:
            _drain(procs)
    _drain(procs)
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", out, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    build_calls(hipcc, verbose)
    return out


def build_calls(hipcc: str, verbose: bool = False) -> str:
    """The binding's native entry points: host code against PyTorch's headers, linked to the library beside it."""
    import torch
    troot = os.path.dirname(torch.__file__)
    cmd = [hipcc, "-x", "c++", os.path.join(CSRC, "tm_calls.cpp"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
           "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}",
           "-I", os.path.join(ROOT, "include"), "-isystem", os.path.join(troot, "include"),
           "-isystem", os.path.join(troot, "include", "torch", "csrc", "api", "include"),
           "-isystem", sysconfig.get_paths()["include"], "-isystem", os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(hipcc))), "include"), "-o", CALLS, "-L", PKG, "-l:libtm_w4.so", "-Wl,-rpath,$ORIGIN",
           "-L", os.path.join(troot, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    if verbose:
        print(" ".join(cmd), flush=True)
    done = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if done.returncode != 0:
        raise RuntimeError(f"hipcc failed on tm_calls.cpp:\n{done.stdout}")
    return CALLS


def _drain(procs):
    while procs:
        src, p = procs.pop(0)
        out, _ = p.communicate()
        noise = "is not a recognized feature for this target"
        out = "\n".join(l for l in out.splitlines() if noise not in l)
        if p.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{out}")
        if out.strip():
            print(out, file=sys.stderr)


if __name__ == "__main__":
    print(build(verbose=True))
