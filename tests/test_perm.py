"""Tiles whose runs share indices, permuted in LDS by persistent workgroups
(kernel P), for each number of vectors per lane, one and several tiles per
workgroup, one and several B columns, clipped chunks on either side:
through the host emulator, which checks every offset (small problems with
their data against the oracle, large ones a sample of their tiles), and on an
MI355X against the oracle, bit for bit, whole."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as orc

# extents, perm, dtype, the tile the plan takes (None: any, and only with beta 0)
CASES = [
    ((2, 2), (1, 0), "f32", "4x1 to 4x1 vectors=1 tiles=1 "),
    ((4, 3, 6), (1, 0, 2), "f32", "72x1 to 72x1 vectors=1 tiles=1 "),
    ((16, 20, 2), (2, 1, 0), "f32", "160x2 to 20x16 vectors=1 tiles=2 "),
    ((3, 21, 31, 3, 2, 17), (1, 3, 5, 2, 0, 4), "f32", "126x6 to 126x6 vectors=1 tiles=288 "),
    ((9, 34, 2, 23, 2, 7), (0, 2, 4, 1, 5, 3), "f32", "153x4 to 612x1 vectors=1 tiles=322 "),
    ((6, 3, 5, 20), (3, 2, 1, 0), "f32", "900x1 to 10x90 vectors=2 tiles=2 "),
    ((18, 54, 2, 11, 6), (3, 0, 1, 4, 2), "f32", "139x11 to 1529x1 vectors=2 tiles=84 "),
    ((14, 2, 2, 5, 10), (4, 2, 0, 1, 3), "f32", "1400x1 to 5x280 vectors=3 tiles=2 "),
    ((35, 43, 10), (2, 0, 1), "f32", "251x10 to 2510x1 vectors=3 tiles=6 "),
    ((7, 44, 15), (2, 1, 0), "f32", "308x15 to 4620x1 vectors=5 tiles=1 "),
    ((9, 46, 21, 17), (2, 1, 3, 0), "f32", "207x21 to 483x9 vectors=5 tiles=34 "),
    ((3, 5000017), (1, 0), "f32", None),                 # several tiles per workgroup
    ((1254, 2, 5, 1601), (2, 0, 3, 1), "f32", None),
    ((2, 2), (1, 0), "f64", "4x1 to 4x1 vectors=1 tiles=1 "),
    ((3, 21, 31, 3, 2, 17), (1, 3, 5, 2, 0, 4), "f64", "63x3 to 63x3 vectors=1 tiles=1054 "),
    ((6, 2, 7, 38, 40), (1, 0, 2, 3, 4), "f64", "72x1 to 72x1 vectors=1 tiles=1774 "),
    ((2, 36, 2, 3, 2), (4, 3, 2, 1, 0), "f64", "72x12 to 864x1 vectors=2 tiles=1 "),
    ((55, 10, 26), (2, 1, 0), "f64", "55x26 to 26x55 vectors=3 tiles=10 "),
    ((24, 2, 13, 45), (3, 2, 0, 1), "f64", "48x45 to 45x48 vectors=5 tiles=13 "),
    ((24, 26, 26), (2, 0, 1), "f64", "63x26 to 1638x1 vectors=5 tiles=10 "),
]
# the cases whose problem, its last index cut short, is kernel P's too
CUT_TAKEN = [
    ((4, 3, 6), "f32"), ((3, 21, 31, 3, 2, 17), "f32"), ((9, 34, 2, 23, 2, 7), "f32"),
    ((6, 3, 5, 20), "f32"), ((18, 54, 2, 11, 6), "f32"), ((14, 2, 2, 5, 10), "f32"),
    ((7, 44, 15), "f32"), ((9, 46, 21, 17), "f32"), ((3, 21, 31, 3, 2, 17), "f64"),
    ((6, 2, 7, 38, 40), "f64"),
]
MODES = [(1.0, 0.0), (-0.3, 1.25)]


def _rand(rng, n, dtype):
    return (rng.integers(-(1 << 20), 1 << 20, size=n) / float(1 << 20)).astype(
        np.float32 if dtype == "f32" else np.float64)


def _ids(v):
    return "x".join(map(str, v)) if isinstance(v, tuple) else str(v)


@pytest.mark.parametrize("size,perm,dtype,tile", CASES, ids=_ids)
def test_emulated(size, perm, dtype, tile):
    from emulator import emu
    rng = np.random.default_rng(11)
    for alpha, beta in MODES:
        p = emu.plan(perm, size, alpha, beta, dtype)
        assert f"permute={tile or ''}" in p.describe() or (not tile and beta), p.describe()
        if p.numel > 100000:
            for mis in (0, 1):
                err, msg, _ = emu.run(p, block_stride=53, mis_b=mis)
                assert err == 0, f"{p.describe()}: {msg}"
            continue
        A, B0 = _rand(rng, p.numel, dtype), _rand(rng, p.numel, dtype)
        want = orc.transpose(A, size, perm, alpha, beta, B0 if beta != 0 else None)
        for mis in (0, 1, 3):
            B = B0.copy()
            err, msg, cnt = emu.run(p, A, B, counts=True, mis_b=mis)
            assert err == 0, f"{p.describe()}: {msg}"
            assert (cnt == 1).all() and np.array_equal(B, want), p.describe()


@pytest.mark.gpu
@pytest.mark.parametrize("size,perm,dtype,tile", CASES, ids=_ids)
def test_gpu(size, perm, dtype, tile):
    """Whole tensors, pointers on and off a line, and as blocks of larger tensors."""
    import torch

    from paper_1704_04374_amd import hptt
    rng = np.random.default_rng(12)
    n = int(np.prod(size))
    size_b = [size[p] for p in perm]
    A, B0 = _rand(rng, n + 4, dtype), _rand(rng, n + 4, dtype)
    dA = torch.from_numpy(A).cuda()
    for alpha, beta in MODES:
        p = hptt.create_plan(perm, size, alpha, beta, dtype)
        assert f"permute={tile or ''}" in p.describe() or (not tile and beta), p.describe()
        print(f"[permute] {p.describe()}", flush=True)
        for a, b in ((0, 0), (1, 3), (3, 2)):
            want = B0.copy()
            want[b:b + n] = orc.transpose(A[a:a + n], size, perm, alpha, beta,
                                          B0[b:b + n] if beta != 0 else None)
            dB = torch.from_numpy(B0).cuda()
            p.exec(dA[a:a + n], dB[b:b + n])
            assert np.array_equal(dB.cpu().numpy(), want), (p.describe(), a, b)
    # the last index of A and of B cut short: the rest of B stays as it was
    cut = tuple(s - 1 if d == len(size) - 1 else s for d, s in enumerate(size))
    cut_b = [cut[q] for q in perm]
    p = hptt.create_plan(perm, cut, 1.5, 0.5, dtype, outer_size_a=size, outer_size_b=size_b)
    print(f"[permute] {p.describe()}", flush=True)
    assert ("permute=" in p.describe()) == ((size, dtype) in CUT_TAKEN)
    want = orc.transpose_outer(A[:n], cut, perm, size, size_b, 1.5, 0.5, B0[:n])
    dB = torch.from_numpy(B0[:n].copy()).cuda()
    p.exec(dA[:n], dB)
    assert np.array_equal(dB.cpu().numpy(), want), (p.describe(), cut_b)


@pytest.mark.parametrize("size,perm,dtype,beta,taken", [
    ((5, 6820, 2, 3, 2, 2, 2), (0, 4, 3, 2, 6, 5, 1), "f32", 0.5, False),    # 20 us, kernel T 12
    ((2, 512, 128, 4), (3, 0, 2, 1), "f64", 0.5, False),
    ((5, 6820, 2, 3, 2, 2, 2), (0, 4, 3, 2, 6, 5, 1), "f32", 0.0, True),     # B not read
    ((9, 46, 21, 17), (2, 1, 3, 0), "f32", 0.5, True),                       # below 1 MiB
    ((304944, 5), (1, 0), "f64", 1.0, False),                                # 3 vectors, 11.6 MiB
    ((24944, 5), (1, 0), "f64", 1.0, True),
])
def test_many_vectors_with_b_read(size, perm, dtype, beta, taken):
    """Tiles of five vectors per lane are not taken from 1 MiB on where B is read,
    tiles of three not from 6 MiB on."""
    from paper_1704_04374_amd import hptt
    p = hptt.create_plan(perm, size, 1.0, beta, dtype)
    assert ("permute=" in p.describe()) == taken, p.describe()
