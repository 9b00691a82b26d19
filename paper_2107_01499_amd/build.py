"""Compile the HIP sources under csrc/ into paper_2107_01499_amd/lib/libbagua_hip.so for gfx950, and csrc/native.cpp, the
host path of the binding, into the Python extension lib/_native-torch<version>.<Python's suffix>.  The library needs hipcc; the
extension needs a C++ compiler and the headers of Python and torch, and the package works without it.

Flags that are part of the numerical contract: -ffp-contract=off (no fused multiply-add, every
operation rounds once), no fast-math (correctly rounded division, IEEE denormals), and packed fp32
instructions disabled.
"""
import os
import shutil
import subprocess
import sys
import sysconfig
import warnings

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIBDIR = os.path.join(HERE, "lib")
LIB = os.path.join(LIBDIR, "libbagua_hip.so")
SOURCES = ["api.hip", "batch.hip", "minmax.hip", "sign.hip", "ring.hip", "flatten.hip", "fused.hip", "optim.hip", "topk.hip", "probe.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CXX = os.environ.get("CXX", "g++")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off",
         "-fno-fast-math", "-fhip-fp32-correctly-rounded-divide-sqrt", "-fno-gpu-flush-denormals-to-zero",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wextra", "-Wno-unused-parameter",
         "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd))
    res = subprocess.run(cmd, stderr=subprocess.PIPE, text=True)
    # the host pass does not know the gfx950 feature name of the packed-fp32 switch and says so once per file
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
    if err.strip():
        sys.stderr.write(err + "\n")
    if res.returncode != 0:
        raise subprocess.CalledProcessError(res.returncode, cmd)


def native_path(libdir=LIBDIR, torch_version=None):
    """The host extension for this Python and its torch.  It uses their C++ types, so one that was built for others must not
    be loaded: the name tells them apart, and after a change of either there is none until it is built again."""
    import torch
    return os.path.join(libdir, "_native-torch%s%s" % (torch_version or torch.__version__, sysconfig.get_config_var("EXT_SUFFIX")))


def _native_dirs():
    from importlib.util import find_spec
    torch_dir = find_spec("torch").submodule_search_locations[0]
    return sysconfig.get_paths()["include"], os.path.join(torch_dir, "include"), os.path.join(torch_dir, "lib")


def native_lacks():
    """What the extension cannot be built without and is not there, or None."""
    python, torch, _ = _native_dirs()
    if shutil.which(CXX) is None:
        return "the C++ compiler " + CXX
    for header in (os.path.join(python, "Python.h"), os.path.join(torch, "torch", "csrc", "autograd", "python_variable.h")):
        if not os.path.exists(header):
            return header
    return None


def build_native(verbose=False, libdir=LIBDIR):
    """The host extension: plain C++ against the headers of this Python and its torch.  Where they are missing there is none,
    nor an older one."""
    os.makedirs(libdir, exist_ok=True)
    out, lacks = native_path(libdir), native_lacks()
    if lacks:
        if os.path.exists(out):
            os.remove(out)
        warnings.warn("the binding's host extension is not built, %s is missing; calls take the general path" % lacks, RuntimeWarning)
        return None
    python, torch, lib = _native_dirs()
    _run([CXX, "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall", "-Wextra",
          "-I" + os.path.join(ROOT, "include"), "-isystem", python,
          "-isystem", torch, "-isystem", os.path.join(torch, "torch", "csrc", "api", "include"),
          os.path.join(CSRC, "native.cpp"), "-L" + lib, "-Wl,-rpath," + lib, "-ltorch_python", "-ltorch_cpu", "-lc10", "-o", out], verbose)
    return out


def build(verbose=False, extra=(), out=LIB):
    """Compile every source to an object (in parallel), then link the shared library; the host extension beside it."""
    from concurrent.futures import ThreadPoolExecutor
    os.makedirs(os.path.dirname(out), exist_ok=True)
    objdir = out + ".obj"
    os.makedirs(objdir, exist_ok=True)
    compile_flags = [f for f in FLAGS if f != "-shared"]

    def compile_one(src):
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        _run([HIPCC] + compile_flags + list(extra) + ["-c", os.path.join(CSRC, src), "-o", obj], verbose)
        return obj

    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as pool:
        native = pool.submit(build_native, verbose, os.path.dirname(out))
        objs = list(pool.map(compile_one, SOURCES))
    _run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC"] + objs + ["-o", out], verbose)
    native.result()
    return out


if __name__ == "__main__":
    print(build(verbose=True, extra=sys.argv[1:]))
