"""Builds libplic.so (HIP kernels + C ABI) in-tree for gfx950 with hipcc, and
_native.so (the torch functions over that ABI, host code) with the host compiler."""
from __future__ import annotations

import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libplic.so")
NATIVE = os.path.join(PKG, "_native.so")
BUILD = os.path.join(os.path.dirname(PKG), "_build")
SOURCES = ["plic_offset.hip", "plic_curvature.hip", "plic_bench.hip", "plic_abi.cpp"]
PARTS = {"plic_curvature.hip": 5}   # objects of a source, compiled with -DPLIC_PART=0, 1, ...
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"
# Packed FP32 (v_pk_*_f32) is disabled for all device code.
FLAGS = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}", "-Wall",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         # keep the execution mask's restore at the end of each inner branch:
         # without it, register reloads that the allocator puts there run for the
         # branch's lanes only, and the others go on with a stale value
         "-Xarch_device", "-mllvm=-amdgpu-remove-redundant-endcf=0"]


def _native_object():
    """The command that compiles plic_torch.cpp, and what links it."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension

    obj = os.path.join(BUILD, "plic_torch.o")
    # packaged headers as system headers: their warnings are not ours
    inc = [f for p in cpp_extension.include_paths() + [sysconfig.get_paths()["include"], "/opt/rocm/include"]
           for f in ("-isystem", p)]
    compile_ = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
                f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", *inc,
                "-c", os.path.join(CSRC, "plic_torch.cpp"), "-o", obj]
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    link = [os.environ.get("CXX", "g++"), "-shared", "-fPIC", obj, "-L" + PKG, "-lplic", "-L" + lib, "-ltorch_python",
            "-ltorch", "-ltorch_cpu", "-lc10", "-lc10_hip", "-Wl,-rpath,$ORIGIN", "-Wl,-rpath," + lib]
    return compile_, link


def build_library(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    native, native_link = _native_object()
    if verbose:
        print(" ".join(native), flush=True)
    procs = [("plic_torch.cpp", subprocess.Popen(native, stdout=subprocess.PIPE, stderr=subprocess.STDOUT))]
    objs = []
    for src in SOURCES:
        for part in range(PARTS.get(src, 1)):
            obj = os.path.join(BUILD, f"{src.rsplit('.', 1)[0]}_{part}.o")
            objs.append(obj)
            cmd = [HIPCC, *FLAGS, *([f"-DPLIC_PART={part}"] if src in PARTS else []), "-c", os.path.join(CSRC, src), "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)))
    failed = []
    for src, p in procs:
        out, _ = p.communicate()
        text = out.decode(errors="replace")
        # hipcc's host pass does not know the packed-fp32 feature: harmless
        lines = [ln for ln in text.splitlines() if "packed-fp32-ops" not in ln and ln.strip()]
        if p.returncode != 0:
            failed.append(src)
            print("\n".join(lines), file=sys.stderr)
        elif verbose and lines:
            print("\n".join(lines))
    if failed:
        raise RuntimeError(f"hipcc failed for {failed}")
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "-shared", "-fPIC", f"--offload-arch={ARCH}", "-o", tmp, *objs,
           "-Wl,-rpath,/opt/rocm/lib"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    tmp = NATIVE + ".tmp"
    cmd = [*native_link, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, NATIVE)
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))
