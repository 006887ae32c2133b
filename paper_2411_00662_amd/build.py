"""Builds libmonta.so (HIP, gfx950) in-tree with hipcc, which cross-compiles without a GPU, and _host.so with the host compiler."""
from __future__ import annotations

import os
import subprocess
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
SRC = os.path.join(PKG, "csrc", "monta.hip")
DEPS = [SRC, os.path.join(PKG, "csrc", "monta_kernels.hpp"), os.path.join(PKG, "csrc", "monta_planner.hpp"),
        os.path.join(ROOT, "include", "monta.h")]
LIB = os.path.join(PKG, "libmonta.so")
HOST_SRC = os.path.join(PKG, "csrc", "host.cpp")
HOST = os.path.join(PKG, "_host.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # keep the compiler from forming packed fp32 instructions out of scalar float code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # the first arguments of a kernel come in registers instead of by a load at its start, which takes 0.25 us (MI355X: a kernel of
    # one load and one store 2.68 -> 2.44 us; 64 tokens, 8 experts, whole step 8.21 -> 7.98, gate of 600 x 1024 4.03 -> 3.76)
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
    "-Wall", "-Wextra",
]


def build(force: bool = True, verbose: bool = False) -> str:
    """Compile the library and the native half of the binding.  With force=False what is up to date is kept."""
    build_host(force, verbose)
    if not force and os.path.exists(LIB) and all(os.path.getmtime(LIB) >= os.path.getmtime(d) for d in DEPS):
        return LIB
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *HIPCC_FLAGS, "-Rpass-analysis=kernel-resource-usage", "-I" + os.path.join(ROOT, "include"),
           "-o", LIB, SRC]
    res = subprocess.run(cmd, capture_output=True, text=True)
    failed = res.returncode != 0
    if verbose or failed:
        print(" ".join(cmd))
        print(res.stdout)
        print("\n".join(l for l in res.stderr.splitlines() if failed or "remark:" not in l))
    if failed:
        raise RuntimeError("hipcc failed building libmonta.so")
    spills = scratch_users(res.stderr)
    if spills:
        # a kernel that spills registers to scratch memory still computes the right thing, many times slower (an
        # innocent-looking edit of the expert kernel once did that): refuse the build rather than ship it
        os.remove(LIB)
        raise RuntimeError("kernels spill registers to scratch: " + ", ".join(f"{k} ({v} B/lane)" for k, v in spills))
    return LIB


def build_host(force: bool = True, verbose: bool = False) -> str:
    """Compile the native half of the binding against torch's headers."""
    deps = [HOST_SRC, os.path.join(ROOT, "include", "monta.h")]
    if not force and os.path.exists(HOST) and all(os.path.getmtime(HOST) >= os.path.getmtime(d) for d in deps):
        return HOST
    import torch
    torch_dir = os.path.dirname(torch.__file__)
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall", "-Wextra",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-I" + os.path.join(ROOT, "include"),
           "-isystem", os.path.join(torch_dir, "include"), "-isystem", sysconfig.get_paths()["include"], "-o", HOST, HOST_SRC,
           "-L" + os.path.join(torch_dir, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if verbose or res.returncode != 0:
        print(" ".join(cmd))
        print(res.stdout, res.stderr)
    if res.returncode != 0:
        raise RuntimeError("the host compiler failed building _host.so")
    return HOST


def scratch_users(remarks: str):
    """(kernel, bytes per lane) for every kernel whose resource-usage remark reports scratch memory."""
    out, name = [], None
    for line in remarks.splitlines():
        if "Function Name:" in line:
            name = line.split("Function Name:")[1].split("[")[0].strip()
        elif "ScratchSize [bytes/lane]:" in line and name:
            n = int(line.split("ScratchSize [bytes/lane]:")[1].split("[")[0].strip())
            if n > 0:
                out.append((name, n))
    return out


if __name__ == "__main__":
    print(build(verbose=True))
