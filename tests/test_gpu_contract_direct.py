"""The direct contraction kernel on an MI355X at the edges of its blocks (128
rows, 64 columns, slices of 8 or 16 contracted positions), in each order its
operands are staged in, against the contraction oracle: every element within
(k + 2) u (|alpha| sum |A||B| + |beta| |C|), the bound of a dot product summed
in any order."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from oracle import contract as oc
from paper_1704_04374_amd.contraction import Contraction

pytestmark = pytest.mark.gpu

NP = {"f32": np.float32, "f64": np.float64}

CASES = [
    # rows of A lead with C's stride-1 mode; rows, columns and slices around a block
    ("mnq=mkq*kn", dict(m=43, q=3, n=63, k=7)),
    ("mnq=mkq*kn", dict(m=64, q=2, n=64, k=16)),
    ("mnq=mkq*kn", dict(m=43, q=3, n=65, k=17)),
    ("mnq=mkq*kn", dict(m=1, q=129, n=1, k=1)),
    # A leads with a contracted mode, B with a column
    ("mnq=kmq*nk", dict(m=33, q=5, n=70, k=9)),
    # A leads with another row mode than C: 8, 3 x 5 and 9 positions staged side by side
    ("mnq=qkm*kn", dict(m=17, q=8, n=20, k=8)),
    ("mnqr=qrkm*kn", dict(m=35, q=3, r=5, n=10, k=15)),
    ("mnq=qmk*kn", dict(m=5, q=9, n=66, k=18)),
    ("abcd=aebf*dfce", dict(a=13, b=11, c=7, d=10, e=3, f=6)),
    # roles swapped (C's stride-1 mode is B's), a batch mode
    ("nmq=mkq*kn", dict(m=20, q=7, n=37, k=11)),
    ("mnlq=mlkq*knl", dict(m=10, q=13, n=9, k=5, l=3)),
]


def _problem(spec, ext, dtype, alpha, beta):
    c, ab = spec.split("=")
    a, b = ab.split("*")
    p = Contraction(c, a, [ext[m] for m in a], b, [ext[m] for m in b], alpha, beta, dtype)
    return p, c, a, b


def _data(rng, modes, ext, dtype):
    return rng.uniform(-1, 1, int(np.prod([ext[m] for m in modes]))).astype(NP[dtype])


@pytest.mark.parametrize("spec,ext", CASES, ids=lambda v: v if isinstance(v, str) else
                         "x".join(map(str, v.values())))
def test_block_edges(spec, ext):
    rng = np.random.default_rng(7)
    for dtype in ("f32", "f64"):
        for alpha, beta in ((1.0, 0.0), (-0.75, 1.25)):
            p, c, a, b = _problem(spec, ext, dtype, alpha, beta)
            print(f"[direct] {p.describe()} beta={beta}", flush=True)
            assert p.describe().endswith("direct")
            A, B, C = (_data(rng, m, ext, dtype) for m in (a, b, c))
            dA, dB, dC = (torch.from_numpy(x).cuda() for x in (A, B, C))
            if beta == 0:
                dC.fill_(float("nan"))     # never read
            p.exec(dA, dB, dC)
            got = dC.cpu().numpy().astype(np.float64)
            sa, sb = p.size_a, p.size_b
            exact = oc.contract(A, a, sa, B, b, sb, c, alpha, beta, C)
            mag = oc.magnitude(A, a, sa, B, b, sb, c, alpha, beta, C)
            assert (np.abs(got - exact) <= oc.error_bound(mag, p.info["gemm_k"], dtype)).all()


def test_large_result_and_overlapping_tensors():
    """C of 64 MiB and more, written non-temporally; and C on top of A, which
    the transpositions serve because they copy A first."""
    ext = dict(m=24, q=24, n=96, k=5, r=152)
    p, c, a, b = _problem("mnqr=qkmr*kn", ext, "f64", 1.0, 0.0)
    assert p.describe().endswith("direct")
    A, B = (torch.rand(int(np.prod([ext[m] for m in s])), dtype=torch.float64, device="cuda")
            for s in (a, b))
    C = torch.empty(int(np.prod([ext[m] for m in c])), dtype=torch.float64, device="cuda")
    assert C.numel() * 8 >= 64 << 20
    print(f"[direct] {p.describe()}", flush=True)
    p.exec(A, B, C)
    t = A.view(ext["r"], ext["m"], ext["k"], ext["q"]).permute(0, 3, 1, 2)   # r q m k
    want = torch.zeros(ext["r"], ext["q"], ext["n"], ext["m"], dtype=torch.float64, device="cuda")
    bt = B.view(ext["n"], ext["k"])
    for k in range(ext["k"]):
        want += t[:, :, None, :, k] * bt[None, None, :, k, None]
    assert (C.view_as(want) - want).abs().max() <= (ext["k"] + 2) * 2.0 ** -53 * ext["k"]
    ext = dict(m=16, q=8, n=4, k=4)
    p, c, a, b = _problem("mnq=qkm*kn", ext, "f64", 1.0, 0.0)
    assert p.describe().endswith("direct") and p.info["transpose_a"]
    rng = np.random.default_rng(3)
    A, B = _data(rng, a, ext, "f64"), _data(rng, b, ext, "f64")
    dA = torch.from_numpy(A).cuda()
    p.exec(dA, torch.from_numpy(B).cuda(), dA)
    exact = oc.contract(A, a, p.size_a, B, b, p.size_b, c)
    mag = oc.magnitude(A, a, p.size_a, B, b, p.size_b, c)
    assert (np.abs(dA.cpu().numpy() - exact) <= oc.error_bound(mag, 4, "f64")).all()
