"""Build libflexgemm.so (HIP kernels + C ABI) for gfx950, in-tree, with hipcc, and the binding's native
marshalling (csrc/fastcall.cpp) with the host compiler and the headers of the torch it will be used with; without either the
binding marshals with ctypes.

Objects go to ``_build/`` at the repository root; the shared library is written next to this
file so that it travels with the package.  ``python -m paper_2009_12263_amd.build`` rebuilds.
"""
from __future__ import annotations

import concurrent.futures as cf
import glob
import os
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libflexgemm.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CXX = os.environ.get("CXX", "g++")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-inline-asm",
         "-Wno-unused-command-line-argument",
         # keep the compiler from forming packed-FP32 instructions: some of their forms have given
         # wrong results on this hardware, with no error, in ways tests do not reliably show
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _stale(target: str, deps) -> bool:
    if not os.path.exists(target):
        return True
    t = os.path.getmtime(target)
    return any(os.path.getmtime(d) > t for d in deps)


def _compile(src: str, force: bool) -> str:
    obj = os.path.join(OBJ, os.path.basename(src)[:-4] + ".o")
    deps = [src] + glob.glob(os.path.join(CSRC, "*.hpp")) + glob.glob(os.path.join(ROOT, "include", "*.h"))
    if force or _stale(obj, deps):
        cmd = [HIPCC] + FLAGS + ["-c", src, "-o", obj]
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        out = "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l)
        if r.returncode != 0:
            raise RuntimeError("hipcc failed on %s:\n%s" % (src, out))
        if out.strip():
            sys.stderr.write(out + "\n")
    return obj


def _build_fastcall(force: bool) -> None:
    import torch
    from .binding import FASTCALL_PATH
    src = os.path.join(CSRC, "fastcall.cpp")
    if not (force or _stale(FASTCALL_PATH, [src] + glob.glob(os.path.join(ROOT, "include", "*.h")))):
        return
    base = os.path.dirname(torch.__file__)
    lib = os.path.join(base, "lib")
    tmp = FASTCALL_PATH + ".tmp.%d" % os.getpid()
    cmd = [CXX, "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall", src, "-o", tmp,
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
           "-isystem", os.path.join(base, "include"), "-isystem", os.path.join(base, "include", "torch", "csrc", "api", "include"),
           "-isystem", sysconfig.get_paths()["include"],
           "-L" + lib, "-Wl,-rpath," + lib, "-ltorch_python", "-ltorch_cpu", "-lc10", "-lpthread"]
    try:
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        built, said = r.returncode == 0, r.stdout
    except OSError as e:
        built, said = False, str(e)
    if built:
        os.replace(tmp, FASTCALL_PATH)
    else:
        if os.path.exists(FASTCALL_PATH):        # built from older sources
            os.remove(FASTCALL_PATH)
        said = "%s failed on %s, the binding will use ctypes:\n%s" % (CXX, src, said)
    if said.strip():
        sys.stderr.write(said + "\n")


def build(force: bool = False, jobs: int = 8) -> str:
    os.makedirs(OBJ, exist_ok=True)
    srcs = sources()
    with cf.ThreadPoolExecutor(max_workers=min(jobs, len(srcs) + 1)) as ex:
        fastcall = ex.submit(_build_fastcall, force)
        objs = list(ex.map(lambda s: _compile(s, force), srcs))
        fastcall.result()
    if force or _stale(LIB, objs):
        tmp = LIB + ".tmp.%d" % os.getpid()
        subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs)
        os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(force="--force" in sys.argv))
