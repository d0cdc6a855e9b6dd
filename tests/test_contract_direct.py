"""The direct contraction kernel's planner and index arithmetic on the CPU:
random contractions of every mix of roles, in both types, against the contraction
oracle on whole numbers (exact in any order), with every offset checked, the
blocks of the benchmark contractions at full size, and tensors at the limits of the
32-bit offsets."""
from __future__ import annotations

import ctypes
import os
import re
import subprocess

import numpy as np
import pytest

from emulator import build as emu_build
from oracle import contract as oc
from paper_1704_04374_amd import build


def _library():
    lib = ctypes.CDLL(emu_build.build_direct())
    vp = ctypes.c_void_p
    lib.direct_emulate.argtypes = ([ctypes.c_char_p] * 3 + [vp, ctypes.c_int32] +
                                   [ctypes.c_double] * 2 + [vp] * 4 +
                                   [ctypes.c_int64, ctypes.c_char_p, ctypes.c_size_t])
    lib.direct_emulate.restype = ctypes.c_int64
    return lib


ELEM = {"f32": 4, "f64": 8}
NP = {"f32": np.float32, "f64": np.float64}


@pytest.fixture(scope="module")
def lib():
    return _library()


def _run(lib, a, b, c, ext, dtype, alpha=1.0, beta=0.0, A=None, B=None, C=None, counts=None,
         stride=1):
    e = np.zeros(256, dtype=np.int64)
    for m, n in ext.items():
        e[ord(m)] = n
    msg = ctypes.create_string_buffer(256)
    ptr = [None if x is None else x.ctypes.data for x in (A, B, C, counts)]
    rc = lib.direct_emulate(a.encode(), b.encode(), c.encode(), e.ctypes.data, ELEM[dtype], alpha,
                            beta, *ptr, stride, msg, len(msg))
    return rc, msg.value.decode()


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_random_contractions_match_oracle(lib, dtype):
    rng = np.random.default_rng(1704)
    ran = refused = 0
    while ran < 250:
        modes = "abcdefg"[:int(rng.integers(2, 8))]
        roles = rng.integers(0, 4, size=len(modes))
        if rng.random() < 0.7:
            roles[roles == 3] = 2       # most without batch modes
        t = [[m for m, r in zip(modes, roles) if r in keep] for keep in ((0, 2, 3), (1, 2, 3),
                                                                         (0, 1, 3))]
        if not t[0] or not t[1]:
            continue
        for x in t:
            rng.shuffle(x)
        a, b, c = ("".join(x) for x in t)
        ext = {m: int(rng.choice([1, 2, 3, 5, 8, 9, 17, 33])) for m in modes}
        vol = lambda s: int(np.prod([ext[m] for m in s], dtype=np.int64))
        if vol(a) > 20000 or vol(b) > 20000 or vol(c) > 20000 or vol(modes) > 400000:
            continue
        sa, sb = [ext[m] for m in a], [ext[m] for m in b]
        A, B, C = (rng.integers(-4, 5, size=vol(s)).astype(NP[dtype]) for s in (a, b, c))
        alpha, beta = [(1.0, 0.0), (0.5, -2.0)][ran % 2]
        counts = np.zeros(C.size, dtype=np.uint8)
        got = C.copy()
        rc, msg = _run(lib, a, b, c, ext, dtype, alpha, beta, A, B, got, counts)
        if rc == -1:   # C starts with a batch mode, or is a scalar
            first = next((m for m in c if ext[m] > 1), None)
            assert first is None or (first in a and first in b), (a, b, c, ext)
            refused += 1
            continue
        assert rc == 0, (a, b, c, ext, msg)
        assert (counts == 1).all(), (a, b, c, ext)
        want = oc.contract(A, a, sa, B, b, sb, c, alpha, beta, C)
        assert np.array_equal(got, want), (a, b, c, ext)
        ran += 1
    assert refused < ran


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_workload_blocks(lib, dtype):
    """Offsets of a sample of the blocks of every benchmark contraction."""
    from paper_1704_04374_amd.workloads import CONTRACTIONS
    for w in CONTRACTIONS:
        rc, msg = _run(lib, w.modes_a, w.modes_b, w.modes_c, w.ext(), dtype, stride=max(
            1, w.numel(w.modes_c) // (128 * 64 * 20)))
        assert rc == 0, (w.name, msg)


# A, B or C just under 2^32 bytes of fp64 (the fp32 problem has twice the elements
# of mode w): the largest offsets that 32 bits hold, in each order of staging
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("a,b,c,ext", [
    ("mkw", "kn", "mnw", dict(m=8191, k=31, n=3, w=2113)),
    ("kmw", "nk", "mnw", dict(m=8191, k=31, n=3, w=2113)),
    ("wkm", "kn", "mnw", dict(m=8191, k=31, n=3, w=2113)),
    ("mk", "kwn", "mnw", dict(m=3, k=31, n=8191, w=2113)),
    ("mk", "wnk", "mnw", dict(m=3, k=31, n=8191, w=2113)),
    ("mkw", "kn", "mnw", dict(m=1021, k=2, n=521, w=1008)),
    ("wkm", "nk", "mwn", dict(m=1021, k=2, n=521, w=1008)),
    ("mlkw", "kln", "mnlw", dict(m=1021, k=31, n=5, l=17, w=997)),
])
def test_largest_offsets(lib, a, b, c, ext, dtype):
    ext = dict(ext)
    if dtype == "f32":
        ext["w"] *= 2
    vol = lambda s: int(np.prod([ext[m] for m in s], dtype=np.int64)) * ELEM[dtype]
    largest = max(vol(a), vol(b), vol(c))
    assert 2 ** 32 - 2 ** 26 < largest < 2 ** 32, largest
    blocks = max(1, vol(c) // ELEM[dtype] // (128 * 64))
    rc, msg = _run(lib, a, b, c, ext, dtype, stride=max(1, blocks // 300))
    assert rc == 0, msg
    ext["w"] += 1 + 2 ** 26 // (largest // ext["w"])
    assert max(vol(a), vol(b), vol(c)) >= 2 ** 32
    assert _run(lib, a, b, c, ext, dtype)[0] == -1


def test_waves_that_the_registers_allow():
    """5 waves per SIMD in fp32 and 4 in fp64, without a spill, in every variant of
    the kernel: two registers more cost fp32 a wave, and small products 1.19x."""
    cmd = [build.hipcc(), "-x", "hip", *build.HIP_ONLY, *build.COMMON, "--offload-device-only",
           "-Rpass-analysis=kernel-resource-usage", "-c",
           os.path.join(build.CSRC, "contract_direct.hip"), "-o", os.devnull]
    text = subprocess.run(cmd, stderr=subprocess.PIPE, text=True, check=True).stderr
    name = None
    found = {}
    for line in text.splitlines():
        if m := re.search(r"Function Name: \S*direct_kernelI([fd]\w+?)EEEv", line):
            name = m.group(1)
        elif m := re.search(r"(ScratchSize|Occupancy) \[.*?\]: (\d+)", line):
            found.setdefault(name, {})[m.group(1)] = int(m.group(2))
    assert sorted(n[0] for n in found) == ["d"] * 4 + ["f"] * 2, found
    for n, use in found.items():
        assert use == {"ScratchSize": 0, "Occupancy": 5 if n[0] == "f" else 4}, (n, use)
