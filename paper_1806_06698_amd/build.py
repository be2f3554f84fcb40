"""Build libsyev3.so (HIP, gfx950) in-tree with hipcc, and the Python
binding's native part with the host compiler.

    python -m paper_1806_06698_amd.build

compiles the library's sources under csrc/ into
paper_1806_06698_amd/libsyev3.so, and syev3_binding.cpp, which needs torch's
headers, into paper_1806_06698_amd/_binding.so.  hipcc cross-compiles for
gfx950 without a GPU present.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig
import tempfile

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libsyev3.so")
BINDING = os.path.join(PKG, "_binding.so")

SOURCES = ["syev3_kernels.hip", "syev3_noalloc.hip", "syev3_api.cpp", "syev3_server.cpp"]

ARCH = os.environ.get("SYEV3_OFFLOAD_ARCH", "gfx950")

HIPCC_FLAGS = [
    f"--offload-arch={ARCH}",
    "-O3",
    "-std=c++17",
    "-fPIC",
    # explicit fma() only: results do not depend on where the compiler
    # would have contracted, so every kernel computes bitwise the same
    "-ffp-contract=off",
    # no packed FP32 instructions in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall",
    "-Wno-unused-function",
]


def hipcc() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found (ROCm toolchain required to build libsyev3.so)")


def build(verbose: bool = False) -> str:
    """Compile every source and link libsyev3.so; always rebuilds."""
    cc = hipcc()
    with tempfile.TemporaryDirectory(prefix="syev3_build_") as tmp:
        objs = []
        for src in SOURCES:
            path = os.path.join(CSRC, src)
            obj = os.path.join(tmp, src + ".o")
            cmd = [cc, *HIPCC_FLAGS, "-I", INCLUDE, "-I", CSRC, "-c", path, "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            p = subprocess.run(cmd, stderr=subprocess.PIPE, text=True)
            if p.returncode != 0:
                sys.stderr.write(p.stderr)
                raise RuntimeError(f"hipcc failed on {src}")
            if verbose:
                sys.stderr.write(p.stderr)
            objs.append(obj)
        out_tmp = LIB + ".tmp"
        rocm_lib = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(cc))), "lib")
        cmd = [cc, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", out_tmp, *objs,
               "-L" + rocm_lib, "-Wl,-rpath," + rocm_lib, "-lrocprofiler-sdk-roctx",
               "-lpthread"]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
        os.replace(out_tmp, LIB)
    build_binding(cc, verbose)
    return LIB


def binding_needs() -> str:
    """What this machine lacks to compile the binding ("" if nothing)."""
    if not (shutil.which("g++") or shutil.which("c++")):
        return "a host C++ compiler"
    if not os.path.exists(os.path.join(sysconfig.get_paths()["include"], "Python.h")):
        return "Python's headers"
    try:
        import torch
        from torch.utils import cpp_extension
    except ImportError:
        return "torch"
    if not any(os.path.exists(os.path.join(d, "torch", "csrc", "autograd", "python_variable.h"))
               for d in cpp_extension.include_paths()):
        return "torch's headers"
    return ""


def build_binding(cc: str, verbose: bool = False) -> str | None:
    """Compile the binding (host code only) against the library just built.
    The library and the package work without it: where this machine cannot
    compile it, says so and returns None."""
    if os.path.exists(BINDING):
        os.remove(BINDING)  # never a binding of other sources than the library's
    needs = binding_needs()
    if needs:
        sys.stderr.write(f"{BINDING} is not built (no {needs.removeprefix('a ')} here): calls "
                         "from Python take the slower Python code\n")
        return None
    import torch
    from torch.utils import cpp_extension

    rocm = os.path.dirname(os.path.dirname(os.path.realpath(cc)))
    torch_lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    out_tmp = BINDING + ".tmp"
    cmd = [shutil.which("g++") or "c++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           f'-DSYEV3_TORCH_VERSION="{torch.__version__}"',
           "-I", INCLUDE, *[a for d in cpp_extension.include_paths() for a in ("-isystem", d)],
           "-isystem", os.path.join(rocm, "include"),
           "-isystem", sysconfig.get_paths()["include"],
           os.path.join(CSRC, "syev3_binding.cpp"), "-o", out_tmp,
           "-L" + torch_lib, "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip",
           "-L" + PKG, "-l:" + os.path.basename(LIB), "-Wl,-rpath,$ORIGIN",
           "-Wl,-rpath," + torch_lib]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(out_tmp, BINDING)
    return BINDING


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
