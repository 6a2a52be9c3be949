"""Compile the HIP library (csrc/wht_affine.hip) for gfx950 into libwht_affine.so, and the tensor calls'
marshalling (csrc/torch_marshal.cpp) into the extension module _torch_marshal.so, in-tree.

hipcc cross-compiles without a GPU; the extension module takes the host compiler and torch's headers.
Run as `python -m paper_2603_08343_amd.build`.
"""
import importlib.metadata
import importlib.util
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "csrc", "wht_affine.hip")
LIB = os.path.join(HERE, "libwht_affine.so")
# bench-only object (a plain copy kernel): not part of the layer's ABI, never loaded by the binding
COPY_SRC = os.path.join(HERE, "csrc", "copy_bench.hip")
COPY_LIB = os.path.join(HERE, "libwht_copybench.so")
# debug build of the layer's library for one GPU test: after every LDS read the thread overwrites
# what it read with NaN, so that a read that comes before its data (a missing barrier or wait) shows
# up as NaN; carries the widths 512, 4096, 8192, 16384, 768, 3072, 6144 and 12288 only
POISON_LIB = os.path.join(HERE, "libwht_affine_poison.so")

# host code only: the tensor calls' checks and allocations (no device code, no HIP headers)
MARSHAL_SRC = os.path.join(HERE, "csrc", "torch_marshal.cpp")
MARSHAL_LIB = os.path.join(HERE, "_torch_marshal.so")

# host code only, loaded by tests: the rules of dispatch, so that a test finds the sizes at which the kernels change
ROUTE_SRC = os.path.join(HERE, "csrc", "route_query.cpp")
ROUTE_LIB = os.path.join(HERE, "libwht_route.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # packed float32 VALU forms are kept out of the generated code on the test machines.  The
    # feature belongs to the device target; the driver offers no way to pass a cc1 option to the
    # device pass alone, so the host pass sees it too and says it does not know it (filtered below).
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # matrix-core results are consumed by vector ALU code: have them written to VGPRs directly
    "-mllvm", "-amdgpu-mfma-vgpr-form=1",
    "-Wall", "-Wno-unused-function",
]
HEADER = os.path.join(os.path.dirname(HERE), "include", "wht_affine.h")
SOURCES = [SRC, HEADER] + [os.path.join(HERE, "csrc", f) for f in ("wht_device.h", "wht_plan.h", "wht_route.h", "wht_validate.h")]


def build(verbose: bool = False, extra=()) -> str:
    _compile(COPY_SRC, COPY_LIB, verbose, extra)
    _compile(SRC, POISON_LIB, verbose, (*extra, "-DWHT_POISON_LDS"))
    _compile_marshal(verbose)
    _compile_route(verbose)
    return _compile(SRC, LIB, verbose, extra)


def _compile_marshal(verbose: bool) -> None:
    torch_dir = os.path.dirname(importlib.util.find_spec("torch").origin)
    lib_dir = os.path.join(torch_dir, "lib")
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           "-isystem", os.path.join(torch_dir, "include"),
           "-isystem", os.path.join(torch_dir, "include", "torch", "csrc", "api", "include"), "-isystem", sysconfig.get_paths()["include"],
           f'-DWHT_TORCH_VERSION="{importlib.metadata.version("torch")}"',
           "-o", MARSHAL_LIB, MARSHAL_SRC, "-L" + lib_dir, "-ltorch_python", "-ltorch_hip", "-ltorch_cpu", "-lc10"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)


def _compile_route(verbose: bool) -> None:
    cmd = [os.environ.get("CXX", "g++"), "-O1", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wextra", "-o", ROUTE_LIB, ROUTE_SRC]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)


def _compile(src: str, lib: str, verbose: bool, extra=()) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *HIPCC_FLAGS, *extra, "-o", lib, src]
    if verbose:
        print(" ".join(cmd), flush=True)
    proc = subprocess.run(cmd, stderr=subprocess.PIPE, text=True)
    noise = "'-packed-fp32-ops' is not a recognized feature for this target"
    for line in proc.stderr.splitlines():
        if noise not in line:
            print(line, file=sys.stderr)
    if proc.returncode != 0:
        raise subprocess.CalledProcessError(proc.returncode, cmd)
    return lib


def ensure_built(verbose: bool = False) -> str:
    """For harnesses (tests, smoke check, benchmark): compile only if nothing has been built yet.
    The binding itself never builds: a missing library is an error there."""
    if not all(os.path.exists(lib) for lib in (LIB, COPY_LIB, POISON_LIB, MARSHAL_LIB, ROUTE_LIB)):
        build(verbose=verbose)
    elif any(os.path.getmtime(f) > os.path.getmtime(MARSHAL_LIB) for f in (MARSHAL_SRC, HEADER)):
        raise RuntimeError(f"{MARSHAL_LIB} is older than its source: run `python -m paper_2603_08343_amd.build`")
    elif any(os.path.getmtime(f) > os.path.getmtime(ROUTE_LIB)
             for f in (ROUTE_SRC, os.path.join(HERE, "csrc", "wht_route.h"), os.path.join(HERE, "csrc", "wht_validate.h"), HEADER)):
        raise RuntimeError(f"{ROUTE_LIB} is older than its sources: run `python -m paper_2603_08343_amd.build`")
    elif any(os.path.getmtime(f) > min(os.path.getmtime(LIB), os.path.getmtime(POISON_LIB))
             for f in SOURCES if os.path.exists(f)):
        # a stale binary would be validated and recorded under the new sources' name
        raise RuntimeError(f"{LIB} is older than its sources: run `python -m paper_2603_08343_amd.build`")
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
