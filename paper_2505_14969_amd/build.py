"""Build libstree.so (the C-ABI HIP library) for gfx950 with hipcc, and _host.so (the binding's native half) with the
host compiler against the installed torch, both in-tree.  The library needs neither torch nor the host compiler, and is
there also where _host.so cannot be built."""
from __future__ import annotations

import glob
import os
import shlex
import shutil
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
        raise RuntimeError(f"{os.path.basename(cmd[0])} failed:\n" + err)
    if verbose and err.strip():
        print(err, file=sys.stderr)


def rocm_root() -> str:
    """Where HIP's headers are: ROCM_PATH, beside the compiler that HIPCC names (by a path or a bare name), or /opt/rocm."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    found = os.path.realpath(shutil.which(hipcc) or hipcc)
    for root in (os.environ.get("ROCM_PATH"), os.path.dirname(os.path.dirname(found))):
        if root and os.path.exists(os.path.join(root, "include", "hip", "hip_runtime.h")):
            return root
    return "/opt/rocm"


def host_command():
    """The host compiler's line for _host.so: no device code, the installed torch's headers and libraries."""
    import sysconfig

    import torch
    root = os.path.dirname(os.path.abspath(torch.__file__))
    rocm = rocm_root()
    return [*shlex.split(os.environ.get("CXX", "g++")), "-O2", "-std=c++17", "-fPIC", "-shared", "-DNDEBUG", "-D__HIP_PLATFORM_AMD__=1",
            "-DUSE_ROCM=1", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-Wno-deprecated-declarations",
            "-isystem", os.path.join(root, "include"), "-isystem", sysconfig.get_paths()["include"],
            "-isystem", os.path.join(rocm, "include"), os.path.join(CSRC, "host.cpp"), "-L" + os.path.join(root, "lib"),
            "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]


def build(verbose: bool = False) -> str:
    """Compile every source to an object file (side by side, a few at a time) and link them; the native half of the
    binding beside them (its failure is raised when the library is in its place)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    flags = [f for f in HIPCC_FLAGS if f != "-shared"]
    jobs = max(1, min(8, os.cpu_count() or 1))
    with tempfile.TemporaryDirectory(prefix="stree_build_") as tmp:
        objs = [os.path.join(tmp, os.path.basename(src) + ".o") for src in sources()]
        with ThreadPoolExecutor(max_workers=jobs) as pool:
            host = pool.submit(lambda: _run(host_command() + ["-o", HOST + ".tmp"], verbose))
            list(pool.map(lambda so: _run([hipcc] + flags + ["-c", so[0], "-o", so[1]], verbose), zip(sources(), objs)))
        _run([hipcc] + HIPCC_FLAGS + objs + ["-o", LIB + ".tmp"], verbose)
    os.replace(LIB + ".tmp", LIB)
    host.result()
    os.replace(HOST + ".tmp", HOST)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
