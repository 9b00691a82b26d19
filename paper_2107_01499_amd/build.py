"""Compile the HIP sources under csrc/ into paper_2107_01499_amd/lib/libbagua_hip.so for gfx950, and csrc/native.cpp, the
host path of the binding, into the Python extension lib/_native.so.

Flags that are part of the numerical contract: -ffp-contract=off (no fused multiply-add, every
operation rounds once), no fast-math (correctly rounded division, IEEE denormals), and packed fp32
instructions disabled.
"""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIBDIR = os.path.join(HERE, "lib")
LIB = os.path.join(LIBDIR, "libbagua_hip.so")
NATIVE = os.path.join(LIBDIR, "_native.so")
SOURCES = ["api.hip", "batch.hip", "minmax.hip", "sign.hip", "ring.hip", "flatten.hip", "fused.hip", "optim.hip", "topk.hip", "probe.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
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


def build_native(verbose=False, out=NATIVE):
    """The host extension: plain C++ against the headers of this Python and its torch."""
    import sysconfig
    from importlib.util import find_spec
    os.makedirs(os.path.dirname(out), exist_ok=True)
    torch_dir = find_spec("torch").submodule_search_locations[0]
    lib = os.path.join(torch_dir, "lib")
    _run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall", "-Wextra",
          "-I" + os.path.join(ROOT, "include"), "-isystem", sysconfig.get_paths()["include"],
          "-isystem", os.path.join(torch_dir, "include"), "-isystem", os.path.join(torch_dir, "include", "torch", "csrc", "api", "include"),
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
        native = pool.submit(build_native, verbose, os.path.join(os.path.dirname(out), "_native.so"))
        objs = list(pool.map(compile_one, SOURCES))
        native.result()
    _run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC"] + objs + ["-o", out], verbose)
    return out


if __name__ == "__main__":
    print(build(verbose=True, extra=sys.argv[1:]))
