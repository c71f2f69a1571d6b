"""Builds libpurine_conv.so (HIP kernels + C ABI + executor) for gfx950 with hipcc, in-tree."""
import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libpurine_conv.so")
OBJ_DIR = os.path.join(PKG, "_build")

# -packed-fp32-ops: keep the compiler from forming packed fp32 VALU instructions.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-x", "hip",
         "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function"]


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith((".hip", ".cpp")))


def _compile(src):
    obj = os.path.join(OBJ_DIR, os.path.basename(src) + ".o")
    proc = subprocess.run(["hipcc"] + FLAGS + ["-c", src, "-o", obj], capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in proc.stderr.splitlines() if noise not in l)
    if proc.returncode != 0:
        raise RuntimeError("hipcc failed on %s:\n%s" % (src, err))
    if err.strip():
        print(err)
    return obj


def build_marshal():
    """The native argument marshalling of the Python binding (host code only).

    NDEBUG: pybind11's headers otherwise bring a thread_local counter, and with it a TLS segment. Loading a module with one
    makes every access to the thread_locals of libraries loaded before it (this library's and the HIP runtime's, several
    per launch) take the dynamic linker's slow path: 38.1 instead of 37.1 us for a pass of a single small layer."""
    import sysconfig
    import torch
    tdir = os.path.dirname(torch.__file__)
    out = os.path.join(PKG, "_marshal.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-DNDEBUG", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
                           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
                           "-I" + os.path.join(ROOT, "include"), "-I" + sysconfig.get_paths()["include"],
                           "-isystem", os.path.join(tdir, "include"), "-isystem", "/opt/rocm/include",
                           os.path.join(PKG, "native", "marshal.cpp"), "-o", out,
                           "-L" + PKG, "-l:" + os.path.basename(LIB), "-Wl,-rpath,$ORIGIN",
                           "-L" + os.path.join(tdir, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"])
    return out


def build_library(jobs=4):
    """Compiles every source (always: no up-to-date shortcut) and links the shared library and the binding's module."""
    os.makedirs(OBJ_DIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(_compile, sources()))
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs)
    build_marshal()
    return LIB


if __name__ == "__main__":
    print(build_library())
