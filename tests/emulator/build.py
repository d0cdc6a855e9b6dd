"""Build the test-only host emulator library ``libhptt_emulate.so``.

It compiles ``emulate.cpp`` (host code that runs the kernels' phase functions
with checked memory) together with the library's plan builder and host ABI,
for the host only.  The product library ``libhptt.so`` never contains it.
"""
from __future__ import annotations

import os

from paper_1704_04374_amd import build as lib_build

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
CSRC = os.path.join(ROOT, "paper_1704_04374_amd", "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(HERE, "libhptt_emulate.so")
# the direct contraction kernel's planner and index arithmetic, likewise
DIRECT_LIB = os.path.join(HERE, "libdirect_emulate.so")


def build(verbose: bool = False) -> str:
    _compile([os.path.join(HERE, "emulate.cpp"), os.path.join(CSRC, "plan.cpp"),
              os.path.join(CSRC, "api.cpp")], LIB, verbose)
    build_direct(verbose)
    return LIB


def build_direct(verbose: bool = False) -> str:
    return _compile([os.path.join(HERE, "direct_emulate.cpp"),
                     os.path.join(CSRC, "contract_direct_plan.cpp")], DIRECT_LIB, verbose)


def _compile(srcs, lib, verbose) -> str:
    tmp = f"{lib}.tmp{os.getpid()}"  # one per process: test workers may build at once
    cmd = [lib_build.hipcc(), "-x", "hip", "--offload-host-only", "-O2", "-g", "-std=c++17", "-fPIC",
           "-shared", "-ffp-contract=off", "-Wall", f"-I{INCLUDE}", f"-I{CSRC}", *srcs, "-o", tmp]
    lib_build.run_step(os.path.basename(lib), cmd, verbose)
    os.replace(tmp, lib)
    return lib


if __name__ == "__main__":
    print(build(verbose=True))
