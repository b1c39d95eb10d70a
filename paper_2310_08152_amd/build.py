"""Build libsckv.so (every HIP source under csrc/) for gfx950 with hipcc, and
the native half of the Python binding (csrc/bind.cpp, host code against
torch's headers) with the host compiler.

Objects go to ``_build/`` at the repository root; the shared libraries are
written next to this file.  ``python -m paper_2310_08152_amd.build``.
"""
from __future__ import annotations

import concurrent.futures as cf
import glob
import os
import shutil
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
OUT = os.path.join(PKG, "libsckv.so")
BIND = os.path.join(PKG, "_bind.so")
ARCH = "gfx950"

HIPCC_FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
    # packed fp32 VALU forms are kept out of every kernel
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-I", INCLUDE,
]


def _hipcc() -> str:
    h = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(h):
        raise RuntimeError("hipcc not found")
    return h


def _run(cmd):
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    lines = [ln for ln in r.stdout.splitlines() if "packed-fp32-ops" not in ln]
    return r.returncode, "\n".join(lines)


def _bind_cmd(out):
    """The binding's compile line (torch is found here, not at import)."""
    import sysconfig

    import torch
    tdir = os.path.dirname(torch.__file__)
    cxx = shutil.which("g++") or shutil.which("c++") or _hipcc()
    return [cxx, "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-I", INCLUDE,
            "-isystem", os.path.join(tdir, "include"),
            "-isystem", os.path.join(tdir, "include", "torch", "csrc", "api", "include"),
            "-I", sysconfig.get_paths()["include"],
            "-isystem", os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(_hipcc()))),
                                     "include"),
            os.path.join(CSRC, "bind.cpp"), "-o", out, "-L" + os.path.join(tdir, "lib"),
            "-ltorch_python", "-ltorch_cpu", "-lc10", "-Wl,-rpath," + os.path.join(tdir, "lib")]


def build(verbose: bool = False, jobs: int = 8) -> str:
    hipcc = _hipcc()
    bdir = os.path.join(ROOT, "_build")
    os.makedirs(bdir, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    objs = [os.path.join(bdir, os.path.basename(s)[:-4] + ".o") for s in srcs]

    def compile_one(pair):
        src, obj = pair
        return _run([hipcc, *HIPCC_FLAGS, "-c", src, "-o", obj])

    with cf.ThreadPoolExecutor(max_workers=max(1, jobs)) as ex:
        bind = ex.submit(lambda: _run(_bind_cmd(BIND + ".tmp")))
        results = list(ex.map(compile_one, zip(srcs, objs)))
        rc, out = bind.result()
    if rc != 0:
        raise RuntimeError(f"compiler failed on bind.cpp:\n{out}")
    os.replace(BIND + ".tmp", BIND)
    for (src, _), (rc, out) in zip(zip(srcs, objs), results):
        if verbose and out.strip():
            print(out)
        if rc != 0:
            raise RuntimeError(f"hipcc failed on {os.path.basename(src)}:\n{out}")
    tmp = OUT + ".tmp"
    rc, out = _run([hipcc, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs])
    if rc != 0:
        raise RuntimeError(f"link failed:\n{out}")
    os.replace(tmp, OUT)
    return OUT


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
