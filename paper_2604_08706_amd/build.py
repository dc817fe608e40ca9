"""Build librbpolicy.so (HIP, gfx950 only) and the binding's _marshal module in-tree.

    python -m paper_2604_08706_amd.build         # or: python paper_2604_08706_amd/build.py

Every .hip file under csrc/ is compiled to an object with hipcc and the
objects are linked into paper_2604_08706_amd/librbpolicy.so.  csrc/marshal.cpp,
host code against the torch and Python headers, is compiled with g++ and
linked with the library into paper_2604_08706_amd/_marshal.so; without torch
only the library, which a C program links, is built.  Compiling for gfx950 needs
no GPU, so this runs on any machine with ROCm installed.
"""

import os
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
OBJDIR = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "librbpolicy.so")
MARSHAL = os.path.join(PKG, "_marshal.so")

ARCH = "gfx950"
FLAGS = [
    "-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
    # packed fp32 VALU ops are kept out of every kernel
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
    f"-I{INCLUDE}", f"-I{CSRC}",
]


def hipcc():
    path = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(path):
        raise RuntimeError("hipcc not found (ROCm is required to build librbpolicy.so)")
    return path


def _compile(src, extra):
    obj = os.path.join(OBJDIR, os.path.basename(src) + ".o")
    cmd = [hipcc(), *FLAGS, *extra, "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stderr}")
    noise = [ln for ln in r.stderr.splitlines() if "packed-fp32-ops" not in ln]
    if noise:
        sys.stderr.write("\n".join(noise) + "\n")
    return obj


def _torch_root():
    """Folder of the installed torch, None without one."""
    import importlib.util

    spec = importlib.util.find_spec("torch")
    return None if spec is None else os.path.dirname(spec.origin)


def _run(cmd, what):
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"{what} failed:\n{r.stderr}")


def _compile_marshal():
    """Object of csrc/marshal.cpp."""
    inc = os.path.join(_torch_root(), "include")
    obj = os.path.join(OBJDIR, "marshal.cpp.o")
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(hipcc())))
    _run(["g++", "-O2", "-std=c++17", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
          f"-I{INCLUDE}", f"-I{sysconfig.get_paths()['include']}", "-isystem", inc, "-isystem",
          os.path.join(inc, "torch", "csrc", "api", "include"), "-isystem",
          os.path.join(rocm, "include"), "-c", os.path.join(CSRC, "marshal.cpp"), "-o", obj],
         "g++ on marshal.cpp")
    return obj


def _link_marshal(obj):
    """_marshal.so, next to the library it loads (torch's own are loaded by then)."""
    tmp = MARSHAL + ".tmp"
    _run(["g++", "-shared", obj, f"-L{PKG}", "-l:librbpolicy.so",
          f"-L{os.path.join(_torch_root(), 'lib')}", "-ltorch_python", "-ltorch_cpu", "-lc10_hip",
          "-lc10", "-Wl,-rpath,$ORIGIN", "-o", tmp], "linking _marshal.so")
    os.replace(tmp, MARSHAL)


def build(extra_flags=(), verbose=True):
    """Compile every csrc/*.hip and link librbpolicy.so (its path is returned),
    then, where torch is installed, the _marshal module."""
    os.makedirs(OBJDIR, exist_ok=True)
    srcs = sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))
    workers = min(len(srcs) + 1, max(1, min(8, os.cpu_count() or 1)))
    python = _torch_root() is not None
    with ThreadPoolExecutor(workers) as ex:
        marshal = ex.submit(_compile_marshal) if python else None
        objs = list(ex.map(lambda s: _compile(s, list(extra_flags)), srcs))
    tmp = LIB + ".tmp"
    cmd = [hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, LIB)
    # the library needs neither torch nor g++: it is in place whatever follows
    if python:
        _link_marshal(marshal.result())
    else:
        sys.stderr.write("torch is not installed: _marshal.so, which only the Python binding "
                         "needs, is not built\n")
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build()
