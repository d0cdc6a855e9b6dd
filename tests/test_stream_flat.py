"""The flat walk of kept rows at its edges -- rows as short as one vector, rows
on both sides of the length where an update of B changes its walk, last vectors
of 1 to 3 elements, more rows than one table holds at once -- through the host
emulator and on an MI355X, against the oracle, bit for bit."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as orc

# row length, outer extents (perm reverses them), dtype, plan options
CASES = [
    (4, (5, 3), "f32", {"kernel": "stream", "flat_runs": 1}),
    (5, (3, 7, 2), "f32", {"kernel": "stream", "flat_runs": 1}),
    (5, (31, 67), "f32", {"kernel": "stream", "flat_runs": 1, "max_vec": 2}),
    (7, (41, 53), "f32", {"kernel": "stream", "flat_runs": 1, "max_vec": 1}),
    (17, (3, 5), "f32", {}),
    (19, (40, 7), "f32", {}),
    (63, (9, 5, 7), "f32", {}),
    (79, (11, 13), "f32", {}),
    (81, (11, 13), "f32", {}),      # beyond 320 bytes
    (2049, (3, 2), "f32", {}),
    (18, (33, 65), "f32", {"max_blocks": 2}),
    (2, (7, 9), "f64", {"kernel": "stream", "flat_runs": 1}),
    (9, (19, 31), "f64", {}),
    (39, (5, 7, 3), "f64", {}),
    (41, (5, 7, 3), "f64", {}),
]


def _problem(row, outer, dtype, alpha, beta):
    size = (row, *outer)
    perm = (0, *range(len(outer), 0, -1))
    rng = np.random.default_rng(row)
    npd = np.float32 if dtype == "f32" else np.float64
    n = int(np.prod(size))
    A, B = ((rng.integers(-(1 << 20), 1 << 20, size=n) / float(1 << 20)).astype(npd)
            for _ in range(2))
    return size, perm, A, B, orc.transpose(A, size, perm, alpha, beta, B if beta != 0 else None)


@pytest.mark.parametrize("row,outer,dtype,knobs", CASES, ids=str)
def test_emulated(row, outer, dtype, knobs):
    from emulator import emu
    for alpha, beta in ((1.0, 0.0), (-0.3, 1.25)):
        size, perm, A, B, want = _problem(row, outer, dtype, alpha, beta)
        p = emu.plan(perm, size, alpha, beta, dtype, **knobs)
        assert p.info["kernel"] == "stream" and p.info["flat_runs"] == 1, p.describe()
        err, msg, cnt = emu.run(p, A, B, counts=True)
        assert err == 0, f"{p.describe()}: {msg}"
        assert (cnt == 1).all() and np.array_equal(B, want), p.describe()


@pytest.mark.gpu
@pytest.mark.parametrize("row,outer,dtype,knobs", CASES, ids=str)
def test_gpu(row, outer, dtype, knobs):
    import torch

    from paper_1704_04374_amd import hptt
    for alpha, beta in ((1.0, 0.0), (-0.3, 1.25)):
        size, perm, A, B, want = _problem(row, outer, dtype, alpha, beta)
        p = hptt.create_plan(perm, size, alpha, beta, dtype, **knobs)
        print(f"[flat] {p.describe()}", flush=True)
        n = A.size
        for a, b in ((0, 0), (1, 3)):   # pointers on and off the vector grid
            dA = torch.from_numpy(np.concatenate([A, A[:4]])).cuda()
            dA[a:a + n] = torch.from_numpy(A).cuda()
            dB = torch.zeros(n + 4, dtype=dA.dtype, device="cuda")
            dB[b:b + n] = torch.from_numpy(B).cuda()
            p.exec(dA[a:a + n], dB[b:b + n])
            got = dB.cpu().numpy()
            assert np.array_equal(got[b:b + n], want), (p.describe(), a, b)
            assert not got[:b].any() and not got[b + n:].any()
