"""Build the gfx950 shared library ``libhptt.so`` in-tree with hipcc.

``python -m paper_1704_04374_amd.build`` compiles every source under ``csrc/``
(HIP kernels and the host half of the C ABI) into
``paper_1704_04374_amd/libhptt.so``.  Objects go to ``_build/`` at the
repository root, with the command and the compiler's output of every step
beside them (``<step>.log``).
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess
import sys
import time

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libhptt.so")
# Contractions (transposition - GEMM - transposition) link rocBLAS, so they
# live in a library of their own on top of libhptt.so.
CONTRACT_LIB = os.path.join(PKG, "libhptt_contract.so")
CONTRACT_SOURCES = ["contract.hip", "contract_direct.hip", "contract_direct_plan.cpp"]

ARCH = "gfx950"
# the tile kernel instantiations are split over several files so they compile in parallel
SOURCES = ["tile_matrix.hip", "tile_perm.hip", "tile_f32_fast.hip", "tile_f32_shifted.hip",
           "tile_f32_general.hip", "tile_shared.hip", "tile_direct.hip", "tile_f64.hip", "kernels.hip",
           "yardstick.hip", "api.cpp", "plan.cpp", "autotune.cpp"]

# -ffp-contract=off: alpha*a + beta*b is two roundings and an add, never an
# FMA.  The packed-fp32 feature is switched off for every HIP file.
COMMON = ["-O3", "-std=c++17", "-fPIC", "-ffp-contract=off", "-Wall",
          f"-I{INCLUDE}", f"-I{CSRC}"]
HIP_ONLY = [f"--offload-arch={ARCH}", "-Xclang", "-target-feature", "-Xclang",
            "-packed-fp32-ops"]


def hipcc() -> str:
    path = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(path):
        raise RuntimeError("hipcc not found: the HIP library cannot be built")
    return path


def run_step(name: str, cmd: list, verbose: bool = False) -> None:
    """Run one compiler or linker command and keep its output in
    ``_build/<name>.log``.  A failure is raised with all that is known of it:
    the step, its exit status (negative: ended by that signal), how long it
    ran, the command and the output."""
    os.makedirs(BUILD, exist_ok=True)
    start = time.monotonic()
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True,
                       errors="replace")
    took = time.monotonic() - start
    head = f"{name}: exit status {r.returncode} after {took:.1f} s"
    with open(os.path.join(BUILD, name + ".log"), "w") as f:
        f.write(f"{head}\n{' '.join(cmd)}\n{r.stdout}")
    if verbose:
        print(head, flush=True)
    if r.returncode != 0:
        raise RuntimeError(f"build step {head}\n{' '.join(cmd)}\n{r.stdout}")


def _compile(src: str, verbose: bool = False) -> str:
    obj = os.path.join(BUILD, os.path.basename(src) + ".o")
    cmd = [hipcc(), *COMMON, "-c", os.path.join(CSRC, src), "-o", obj]
    if src.endswith(".hip"):
        cmd[1:1] = ["-x", "hip", *HIP_ONLY]
    else:  # host code only: no device pass
        cmd[1:1] = ["-x", "hip", f"--offload-arch={ARCH}", "--offload-host-only"]
    run_step(os.path.basename(src), cmd, verbose)
    return obj


def _link(objs: list, lib: str, libs: list, verbose: bool) -> None:
    tmp = lib + ".tmp"
    run_step(os.path.basename(lib), [hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs,
                                     "-o", tmp, *libs], verbose)
    os.replace(tmp, lib)


def build(verbose: bool = False) -> str:
    """Compile all sources and link ``libhptt.so`` and the contraction library
    on top of it; return the former's path."""
    sources = SOURCES + CONTRACT_SOURCES
    with cf.ThreadPoolExecutor(max_workers=min(8, len(sources))) as ex:
        objs = list(ex.map(lambda s: _compile(s, verbose), sources))
    _link(objs[:len(SOURCES)], LIB, [], verbose)
    _link(objs[len(SOURCES):], CONTRACT_LIB,
          [f"-L{PKG}", "-lhptt", "-lrocblas", "-Wl,-rpath,$ORIGIN"], verbose)
    if verbose:
        print(f"built {LIB} and {CONTRACT_LIB}", flush=True)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
