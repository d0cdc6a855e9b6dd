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
    ("mnq=mkq*kn", dict(m=43, q=3, n=63, k=37)),    # a third slice in fp32, a fifth in fp64
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


@pytest.mark.parametrize("dtype,m,nt", [("f64", 32, True), ("f64", 24, False), ("f32", 64, False)])
@pytest.mark.parametrize("beta", [0.0, 1.25])
def test_large_result(dtype, m, nt, beta):
    """C of 64 MiB and more: written non-temporally in fp64 where its runs (m
    elements) are whole lines, in either update mode, and with C on a line and
    one element off it, where the stores are ordinary ones."""
    ext = dict(m=m, q=24, n=96, k=5, r=152)
    p, c, a, b = _problem("mnqr=qkmr*kn", ext, dtype, 0.75, beta)
    assert p.describe().endswith(" nt direct" if nt else " direct")
    assert (" nt " in p.describe()) == nt
    print(f"[direct] {p.describe()} beta={beta}", flush=True)
    tdt = torch.float32 if dtype == "f32" else torch.float64
    g = torch.Generator(device="cuda").manual_seed(5)
    A, B, C = (torch.rand(int(np.prod([ext[x] for x in s])) + (s == c), dtype=tdt, device="cuda",
                          generator=g) for s in (a, b, c))
    nc = C.numel() - 1
    assert nc * C.element_size() >= 64 << 20 and C.data_ptr() % 128 == 0
    t = A.double().view(ext["r"], ext["m"], ext["k"], ext["q"]).permute(0, 3, 1, 2)   # r q m k
    prod = torch.zeros(ext["r"], ext["q"], ext["n"], ext["m"], dtype=torch.float64, device="cuda")
    bt = B.double().view(ext["n"], ext["k"])
    for k in range(ext["k"]):
        prod += t[:, :, None, :, k] * bt[None, None, :, k, None]
    u = 2.0 ** (-24 if dtype == "f32" else -53)
    for off in (0, 1):
        got = C.clone() if beta else torch.full_like(C, float("nan"))
        p.exec(A, B, got[off:off + nc])
        want = 0.75 * prod.view(-1)
        if beta:
            want += beta * C[off:off + nc].double()
        # |A|, |B|, |C| <= 1: the bound of (k + 2) u (|alpha| sum |A||B| + |beta| |C|)
        bound = (ext["k"] + 2) * u * (0.75 * ext["k"] + abs(beta))
        assert (got[off:off + nc].double() - want).abs().max() <= bound, off
        rest = got[nc:] if off == 0 else got[:1]
        assert bool((rest == (C[nc:] if off == 0 else C[:1])).all() if beta else rest.isnan().all())


def test_overlapping_tensors():
    """C on top of A, which the transpositions serve because they copy A first."""
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
