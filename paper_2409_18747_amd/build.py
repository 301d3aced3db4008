"""Compile the HIP sources under csrc/ for gfx950 into libcottn.so next to this file, and the binding's C++ half
(csrc/marshal.cpp) against the installed torch into _marshal.so.

Usage: ``python -m paper_2409_18747_amd.build`` or :func:`build`.  hipcc cross-compiles
without a GPU.  Every .hip file is compiled to an object in parallel, then linked.
"""
import concurrent.futures
import glob
import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libcottn.so")
MARSHAL = os.path.join(HERE, "_marshal.so")
OBJ_DIR = os.path.join(HERE, "_build")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function"]


def _compile(src: str) -> str:
    obj = os.path.join(OBJ_DIR, os.path.basename(src) + ".o")
    proc = subprocess.run([HIPCC, *FLAGS, "-c", src, "-o", obj], capture_output=True, text=True)
    # the host pass does not know the packed-fp32 feature and says so; that line is noise
    err = "\n".join(l for l in proc.stderr.splitlines() if "packed-fp32-ops" not in l)
    if proc.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, err))
    if err.strip():
        print(err)
    return obj


def marshal_target() -> str:
    """What _marshal.so is compiled against and says so: it holds the layouts of this torch's and this Python's objects."""
    import torch
    return "torch %s, Python %d.%d" % (torch.__version__, *sys.version_info[:2])


def _build_marshal() -> None:
    import torch
    base = os.path.dirname(torch.__file__)
    tmp = MARSHAL + ".tmp.%d" % os.getpid()
    proc = subprocess.run(
        [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
         '-DCOTTN_BUILT_FOR="%s"' % marshal_target(),
         "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), "-isystem", os.path.join(base, "include"),
         "-isystem", os.path.join(base, "include", "torch", "csrc", "api", "include"),
         # the HIP headers next to the compiler; where that is a wrapper, the usual place
         "-isystem", os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(shutil.which(HIPCC) or HIPCC))), "include"),
         "-isystem", "/opt/rocm/include",
         "-isystem", sysconfig.get_paths()["include"], os.path.join(CSRC, "marshal.cpp"), "-o", tmp,
         "-L" + os.path.join(base, "lib"), "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"],
        capture_output=True, text=True)
    if proc.returncode != 0:
        raise RuntimeError("the compiler failed for marshal.cpp:\n%s" % proc.stderr)
    if proc.stderr.strip():
        print(proc.stderr)
    os.replace(tmp, MARSHAL)


def build(jobs: int = 8) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    sources = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    with concurrent.futures.ThreadPoolExecutor(max_workers=jobs) as pool:
        marshal = pool.submit(_build_marshal)
        objs = list(pool.map(_compile, sources))
        tmp = LIB + ".tmp.%d" % os.getpid()
        subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp], check=True)
        os.replace(tmp, LIB)
        marshal.result()   # the library is there also where this raises, and the binding works with it alone
    return LIB


if __name__ == "__main__":
    print(build())
