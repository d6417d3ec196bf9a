"""Build libstree.so (the C-ABI HIP library) for gfx950 with hipcc, and _host.so (the binding's native half) with the
host compiler against the installed torch, both in-tree."""
from __future__ import annotations

import glob
import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libstree.so")
HOST = os.path.join(HERE, "_host.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-fno-gpu-rdc",
    "-Wno-unused-value", "-Wno-unused-command-line-argument",
    # packed-fp32 forms are kept off for all device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + err)
    if verbose and err.strip():
        print(err, file=sys.stderr)


def host_command():
    """The host compiler's line for _host.so: no device code, the installed torch's headers and libraries."""
    import sysconfig

    import torch
    root = os.path.dirname(os.path.abspath(torch.__file__))
    rocm = os.path.dirname(os.path.dirname(os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")))
    return [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-DNDEBUG", "-D__HIP_PLATFORM_AMD__=1",
            "-DUSE_ROCM=1", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-Wno-deprecated-declarations",
            "-isystem", os.path.join(root, "include"), "-isystem", sysconfig.get_paths()["include"],
            "-isystem", os.path.join(rocm, "include"), os.path.join(CSRC, "host.cpp"), "-L" + os.path.join(root, "lib"),
            "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]


def build(verbose: bool = False) -> str:
    """Compile every source to an object file (side by side, a few at a time) and link them; the native half of the
    binding beside them."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    flags = [f for f in HIPCC_FLAGS if f != "-shared"]
    jobs = max(1, min(8, os.cpu_count() or 1))
    with tempfile.TemporaryDirectory(prefix="stree_build_") as tmp:
        objs = [os.path.join(tmp, os.path.basename(src) + ".o") for src in sources()]
        with ThreadPoolExecutor(max_workers=jobs) as pool:
            host = pool.submit(_run, host_command() + ["-o", HOST + ".tmp"], verbose)
            list(pool.map(lambda so: _run([hipcc] + flags + ["-c", so[0], "-o", so[1]], verbose), zip(sources(), objs)))
            host.result()
        _run([hipcc] + HIPCC_FLAGS + objs + ["-o", LIB + ".tmp"], verbose)
    os.replace(HOST + ".tmp", HOST)
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
