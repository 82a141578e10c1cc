"""Builds librfq.so (the HIP kernels and the C ABI) in-tree for gfx950, and
_rfq_calls.so (the binding's native calls; host code only)."""
import glob
import os
import subprocess
import sysconfig
import tempfile
import warnings
from concurrent.futures import ThreadPoolExecutor

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
REPO_DIR = os.path.dirname(PKG_DIR)
LIB_PATH = os.path.join(PKG_DIR, "librfq.so")
CALLS_PATH = os.path.join(PKG_DIR, "_rfq_calls.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CXX = os.environ.get("CXX", "g++")

# -packed-fp32-ops: no packed fp32 VALU instructions are generated.
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def sources():
    return sorted(glob.glob(os.path.join(PKG_DIR, "csrc", "*.hip")))


def build_calls(verbose=False):
    """Compile csrc_host/ against the installed torch into _rfq_calls.so."""
    import torch
    root = os.path.dirname(torch.__file__)
    inc = os.path.join(root, "include")
    tmp = CALLS_PATH + ".tmp"
    cmd = [CXX, "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
           '-DRFQ_TORCH_VERSION="%s"' % torch.__version__,
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
           "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-isystem", inc, "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"),
           "-isystem", "/opt/rocm/include", "-I", sysconfig.get_paths()["include"],
           "-I", os.path.join(REPO_DIR, "include"),
           os.path.join(PKG_DIR, "csrc_host", "calls.cpp"), "-o", tmp,
           "-L", os.path.join(root, "lib"), "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("_rfq_calls build failed:\n" + res.stderr)
    os.replace(tmp, CALLS_PATH)
    return CALLS_PATH


def build_calls_if_possible(verbose=False):
    """build_calls, or a warning and no module where it does not compile here (no
    g++, torch headers that do not fit): librfq does not need it."""
    try:
        return build_calls(verbose)
    except (ImportError, OSError, RuntimeError) as e:
        if os.path.exists(CALLS_PATH):
            os.remove(CALLS_PATH)
        warnings.warn("the binding's native calls are not built, it makes its calls in Python: %s"
                      % e, RuntimeWarning, stacklevel=2)
        return None


def build(verbose=False, extra_flags=(), out=LIB_PATH):
    """Compile every source under csrc/ into librfq.so and the native calls, or
    only the library into `out` with extra compiler flags (always recompiles)."""
    tmp = out + ".tmp"
    flags = [*FLAGS, *extra_flags]

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, capture_output=True, text=True)
        err = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l)
        if res.returncode != 0:
            raise RuntimeError("librfq build failed:\n" + err)
        if verbose and err.strip():
            print(err)

    with tempfile.TemporaryDirectory() as objs, ThreadPoolExecutor(8) as pool:
        def compile_one(src):
            obj = os.path.join(objs, os.path.basename(src) + ".o")
            run([HIPCC, *flags, "-I", os.path.join(REPO_DIR, "include"),
                 "-I", os.path.join(PKG_DIR, "csrc"), "-c", src, "-o", obj])
            return obj
        run([HIPCC, *flags, "-shared", *pool.map(compile_one, sources()), "-o", tmp])
    os.replace(tmp, out)
    if out == LIB_PATH:
        build_calls_if_possible(verbose)
    return out


if __name__ == "__main__":
    print(build(verbose=True))
