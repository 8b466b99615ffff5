"""Build the HIP library (gfx950) and the binding's native part in-tree: paper_2602_15318_amd/libsparrow.so, _native.so."""
from __future__ import annotations

import glob
import importlib.util
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsparrow.so")
NATIVE = os.path.join(HERE, "_native.so")

# The preload count puts the leading scalar arguments of a kernel into scalar registers at launch: a
# wavefront's first load waits for no load of arguments (0.3 to 0.4 us on kernels of 6 to 13 us).
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-inline-asm",
]


def _run(cmd, verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in res.stdout.splitlines()
                    if "packed-fp32-ops" not in l)   # the host pass does not know the feature
    if res.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed:\n" + out)
    if verbose and out.strip():
        print(out)


def build(verbose: bool = False, extra=()) -> str:
    """Compile every csrc/*.hip into one shared library, and csrc/binding.cpp.  Always recompiles."""
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    _run([hipcc, *HIPCC_FLAGS, *extra, "-o", LIB, *srcs], verbose)
    torch = os.path.dirname(importlib.util.find_spec("torch").origin)
    _run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
          "-isystem", os.path.join(torch, "include"), "-isystem", os.path.join(torch, "include", "torch", "csrc", "api", "include"),
          "-isystem", sysconfig.get_paths()["include"], os.path.join(CSRC, "binding.cpp"), "-o", NATIVE,
          "-L" + os.path.join(torch, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"], verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True, extra=sys.argv[1:]))
