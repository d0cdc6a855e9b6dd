"""Flattened two-dimensional tiles (kernel M) at the edges of each tile shape:
through the host emulator, which checks every offset (small problems with
their data against the oracle, large ones a sample of their tiles), and on an
MI355X against the oracle, bit for bit, whole."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as orc

# extents, perm, dtype, the shape the plan takes; columns and rows one off the
# tile, flattened groups of several indices, batches
CASES = [
    ((33, 70), (1, 0), "f32", "16x64"),
    ((4, 65), (1, 0), "f32", "16x64"),
    ((19, 3, 5, 13), (3, 2, 0, 1), "f32", "16x64"),
    ((7, 9, 11, 40), (3, 1, 0, 2), "f32", "16x64"),
    ((128, 64, 96), (1, 0, 2), "f32", "64x64"),          # whole lines
    ((130, 608, 12), (1, 2, 0), "f32", "64x64"),
    ((800, 224, 6), (1, 0, 2), "f32", "128x32"),
    ((1030, 96, 12), (1, 0, 2), "f32", "32x32"),
    ((5120, 5632), (1, 0), "f32", "128x32"),             # 100 to 180 MiB
    ((257, 97, 185), (1, 0, 2), "f32", "32x128"),        # short rows off the lines
    ((50, 601, 145), (1, 0, 2), "f32", "32x128"),        # sheared
    ((5, 13, 40, 1700), (3, 2, 1, 0), "f32", "64x64"),
    ((113, 3, 331, 47), (3, 1, 0, 2), "f32", "64x64"),
    ((9, 465029), (1, 0), "f32", "16x256"),
    ((16, 67, 4099), (1, 2, 0), "f32", "16x256"),
    ((17, 33), (1, 0), "f64", "16x64"),
    ((31, 65, 3), (1, 0, 2), "f64", "16x64"),
    ((7, 5, 131, 9), (2, 3, 0, 1), "f64", "16x64"),
    ((40, 17, 9), (1, 0, 2), "f64", "32x32"),
    ((11, 400), (1, 0), "f64", "8x128"),
    ((31, 19, 701), (2, 1, 0), "f64", "16x64"),          # sheared
    ((514, 512, 11), (1, 0, 2), "f64", "32x64"),
    ((33, 83, 997), (2, 1, 0), "f64", "32x64"),          # sheared
]
MODES = [(1.0, 0.0), (-0.3, 1.25)]


def _rand(rng, n, dtype):
    return (rng.integers(-(1 << 20), 1 << 20, size=n) / float(1 << 20)).astype(
        np.float32 if dtype == "f32" else np.float64)


def _ids(v):
    return "x".join(map(str, v)) if isinstance(v, tuple) else str(v)


@pytest.mark.parametrize("size,perm,dtype,shape", CASES, ids=_ids)
def test_emulated(size, perm, dtype, shape):
    from emulator import emu
    rng = np.random.default_rng(11)
    for alpha, beta in MODES:
        p = emu.plan(perm, size, alpha, beta, dtype)
        assert f"matrix={shape} " in p.describe(), p.describe()
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


@pytest.mark.parametrize("dtype,shape", [("f32", i) for i in range(8)] + [("f64", i) for i in range(6)])
def test_every_shape_emulated(dtype, shape):
    """Each tile shape on small problems with their data, one off its edges in
    columns and rows, fewer columns and rows than a tile, batches, a sub-block:
    whatever the plan would choose at that size."""
    from emulator import emu
    rng = np.random.default_rng(shape)
    cols, rows = emu.set_shape(emu.plan((1, 0, 2), (40, 40, 3), 1.0, 0.0, dtype), shape)
    for c, r, batch in [(cols, rows, 2), (cols + 1, rows - 1, 2), (2 * cols - 1, 2 * rows + 1, 1),
                        (max(5, cols // 2), rows + 33, 3), (cols + 3, max(3, rows // 3), 3),
                        (2 * cols, rows + 31, 1)]:
        for perm, size in (((1, 0, 2), (c, r, batch)), ((1, 2, 0), (c, r, batch))):
            for alpha, beta in MODES:
                p = emu.plan(perm, size, alpha, beta, dtype)
                if "matrix=" not in p.describe():
                    continue
                emu.set_shape(p, shape)
                A, B0 = _rand(rng, p.numel, dtype), _rand(rng, p.numel, dtype)
                want = orc.transpose(A, size, perm, alpha, beta, B0 if beta != 0 else None)
                for mis in (0, 1, 3):
                    B = B0.copy()
                    err, msg, cnt = emu.run(p, A, B, counts=True, mis_b=mis)
                    assert err == 0, f"{size} {perm}: {msg}"
                    assert (cnt == 1).all() and np.array_equal(B, want), (size, perm, mis)
    # a block of larger tensors: the rest of B is not written
    size, outer_a, outer_b = (cols + 2, rows + 3, 2), (cols + 5, rows + 4, 2), (rows + 7, cols + 2, 3)
    p = emu.plan((1, 0, 2), size, 1.5, 0.5, dtype, outer_size_a=outer_a, outer_size_b=outer_b)
    assert "matrix=" in p.describe(), p.describe()
    emu.set_shape(p, shape)
    A, B0 = _rand(rng, int(np.prod(outer_a)), dtype), _rand(rng, int(np.prod(outer_b)), dtype)
    want = orc.transpose_outer(A, size, (1, 0, 2), outer_a, outer_b, 1.5, 0.5, B0)
    B = B0.copy()
    err, msg, _ = emu.run(p, A, B)
    assert err == 0, msg
    assert np.array_equal(B, want)


@pytest.mark.gpu
@pytest.mark.parametrize("size,perm,dtype,shape", CASES, ids=_ids)
def test_gpu(size, perm, dtype, shape):
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
        assert f"matrix={shape} " in p.describe(), p.describe()
        print(f"[matrix] {p.describe()}", flush=True)
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
    print(f"[matrix] {p.describe()}", flush=True)
    # (too few elements in runs of their own, and a large whole-line problem)
    assert ("matrix=" in p.describe()) == (size not in ((19, 3, 5, 13), (5120, 5632)))
    want = orc.transpose_outer(A[:n], cut, perm, size, size_b, 1.5, 0.5, B0[:n])
    dB = torch.from_numpy(B0[:n].copy()).cuda()
    p.exec(dA[:n], dB)
    assert np.array_equal(dB.cpu().numpy(), want), (p.describe(), cut_b)


@pytest.mark.parametrize("size,perm,dtype,taken", [
    ((2, 23, 134079), (1, 0, 2), "f64", False),     # 2 x 23 of 16 x 64
    ((2, 9909223), (1, 0), "f64", False),           # 2 of 8 columns, 159 MB
    ((2, 398160), (1, 0), "f64", True),             # the same, 6 MB
    ((8, 13, 10, 3179, 15), (1, 2, 0, 3, 4), "f32", False),
    ((8, 12, 17266, 2, 29), (1, 2, 0, 4, 3), "f32", True),   # 8 of 16 columns
    ((2, 48, 8, 93, 2, 16), (5, 0, 1, 3, 2, 4), "f64", False),
])
def test_mostly_empty_tiles(size, perm, dtype, taken):
    """Tiles that the problem leaves mostly empty are taken where it is small."""
    from paper_1704_04374_amd import hptt
    assert ("matrix=" in hptt.create_plan(perm, size, 1.0, 0.0, dtype).describe()) == taken


@pytest.mark.parametrize("size,perm,outer_a,outer_b,dtype,taken", [
    ((16, 8, 128, 8, 32), (3, 0, 1, 4, 2), (20, 10, 129, 12, 35), (10, 17, 11, 35, 130), "f32", False),
    ((141908, 2), (1, 0), (141912, 2), (7, 141911), "f32", False),
    ((8969, 18, 2), (2, 0, 1), (8970, 21, 2), (4, 8970, 18), "f32", False),
    ((2, 4, 69, 245), (1, 3, 2, 0), (6, 4, 73, 250), (6, 250, 73, 4), "f64", False),
    ((8969, 2, 2), (2, 0, 1), (8970, 3, 2), (4, 8970, 2), "f32", True),     # few tiles
])
def test_mostly_empty_tiles_of_blocks(size, perm, outer_a, outer_b, dtype, taken):
    """Blocks of larger tensors, whose two rows (or columns) make a matrix each:
    taken where they are few."""
    from paper_1704_04374_amd import hptt
    p = hptt.create_plan(perm, size, 2.0, 0.5, dtype, outer_size_a=outer_a, outer_size_b=outer_b)
    assert ("matrix=" in p.describe()) == taken, p.describe()


def test_hints_of_every_plan_have_a_kernel():
    """Only whole-line tiles of whole-line rows load non-temporally, sheared and
    narrow ones never: the kernels with that hint that are not built."""
    import re

    from paper_1704_04374_amd import hptt
    from paper_1704_04374_amd.workloads import random_problem
    rng = np.random.default_rng(3)
    seen = set()
    for it in range(1500):
        size, perm = random_problem(rng, max_dims=4, max_numel=1 << 26,
                                    extents=(2, 7, 16, 32, 64, 96, 100, 128, 512, 513, 2048))
        dtype = ("f32", "f64")[it % 2]
        m = re.search(r"matrix=(\d+)x\d+ of .* shear=(\d+) tiles=\d+ hints=(\d)",
                      hptt.create_plan(perm, size, 1.0, 0.0, dtype).describe())
        if not m:
            continue
        cols, shear, hints = map(int, m.groups())
        assert hints in (0, 1, 3)
        assert hints != 3 or (shear == 0 and cols * (4 if dtype == "f32" else 8) % 128 == 0)
        seen.add(hints)
    assert seen == {0, 1, 3}


@pytest.mark.parametrize("size,perm,dtype,fits", [
    ((32771, 32749), (1, 0), "f32", True),          # 2^32 - 2.1 M bytes
    ((32771, 32771), (1, 0), "f32", False),
    ((23167, 23161), (1, 0), "f64", True),
    ((23171, 23173), (1, 0), "f64", False),
    ((1021, 1009, 1033, 3), (1, 2, 0, 3), "f32", True),   # the offsets of one of three matrices
    ((37, 5003, 5779), (2, 1, 0), "f32", True),
])
def test_largest_offsets(size, perm, dtype, fits):
    """Matrices just below 2^32 bytes, whose offsets fill 32 bits: the first and
    the last tile and a sample between; those above are kernel T's."""
    import re

    from emulator import emu
    for beta in (0.0, 1.0):
        p = emu.plan(perm, size, 1.0, beta, dtype)
        m = re.search(r"matrix=.* tiles=(\d+)", p.describe())
        assert bool(m) == fits, p.describe()
        if not m:
            continue
        tiles = int(m.group(1))
        for stride in (max(1, tiles - 1), tiles // 211, tiles // 97):
            for mis in (0, 1):
                err, msg, _ = emu.run(p, block_stride=stride, mis_b=mis)
                assert err == 0, f"{p.describe()}: {msg}"
