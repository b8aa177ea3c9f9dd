"""Builds in-tree: csrc/*.hip -> libbcq_hip.so for gfx950, and csrc/bcq_host.cpp -> _bcq_host, the binding's host code."""
from __future__ import annotations

import glob
import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libbcq_hip.so")
HOST_SOURCE = os.path.join(CSRC, "bcq_host.cpp")
HOST_LIB = os.path.join(HERE, "_bcq_host" + sysconfig.get_config_var("EXT_SUFFIX"))      # (another Python does not see it)

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # keep the compiler from forming packed-fp32 VALU instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # the first plain arguments of a kernel arrive in scalar registers (structs are read from memory as before)
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
    "-Wall", "-Wno-unused-command-line-argument",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def is_stale() -> bool:
    if not os.path.exists(LIB) or host_is_stale():
        return True
    t = os.path.getmtime(LIB)
    deps = sources() + glob.glob(os.path.join(CSRC, "*.hpp")) + glob.glob(os.path.join(ROOT, "include", "*.h"))
    return any(os.path.getmtime(d) > t for d in deps)


def host_is_stale() -> bool:
    """Missing for this Python, older than its source, or built against another torch."""
    import torch
    if not os.path.exists(HOST_LIB):
        return True
    if max(os.path.getmtime(f) for f in (HOST_SOURCE, os.path.join(ROOT, "include", "bcq.h"))) > os.path.getmtime(HOST_LIB):
        return True
    with open(HOST_LIB, "rb") as f:
        return f"built for torch {torch.__version__}\0".encode() not in f.read()


def build(verbose: bool = False) -> str:
    """Compile every kernel file with hipcc (cross-compiles without a GPU): one object per source, side by
    side on the available cores, then one link."""
    import concurrent.futures
    import tempfile
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    compile_flags = [f for f in HIPCC_FLAGS if f != "-shared"]
    with tempfile.TemporaryDirectory(prefix="bcq_build_") as tmp:
        def compile_one(src):
            obj = os.path.join(tmp, os.path.basename(src) + ".o")
            cmd = [hipcc, *compile_flags, "-c", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-o", obj, src]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.run(cmd, check=True)
            return obj
        workers = max(1, min(len(sources()), os.cpu_count() or 1, 8))
        with concurrent.futures.ThreadPoolExecutor(max_workers=workers) as pool:
            objects = list(pool.map(compile_one, sources()))
        link = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-Wno-unused-command-line-argument", "-o", LIB, *objects]
        if verbose:
            print(" ".join(link), flush=True)
        subprocess.run(link, check=True)
    build_host(verbose)
    return LIB


def build_host(verbose: bool = False) -> str:
    """The binding's host code, against the torch that is installed (host compiler, no GPU code)."""
    import torch
    torch_dir = os.path.dirname(torch.__file__)
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
           f'-DBCQ_TORCH_VERSION="{torch.__version__}"', f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-I", os.path.join(ROOT, "include"), "-isystem", os.path.join(torch_dir, "include"), "-isystem", "/opt/rocm/include",
           "-isystem", sysconfig.get_paths()["include"], "-o", HOST_LIB, HOST_SOURCE,
           "-L", os.path.join(torch_dir, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return HOST_LIB


if __name__ == "__main__":
    build(verbose=True)
