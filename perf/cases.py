"""The calls whose speed this library is judged by: what they take, how they
run, and what they must return.

A case is one transposition (Eq. 1, ``hptt.Plan.exec``) or one contraction
(``contraction.Contraction.exec``).  The plan, the contraction's workspace
and the tensors are what a program has in hand before the call; ``run`` is
the call itself.  Sizes are written "48x40x32" (Fortran order, first index
fastest), perms "2,0,1" (perm[k] = A index at position k of B).
"""
from __future__ import annotations

import math

import torch

from paper_1704_04374_amd import contraction, hptt
from paper_1704_04374_amd.workloads import CONTRACTIONS_BY_NAME, sweep57

TORCH = {"f32": torch.float32, "f64": torch.float64}
ELEM = {"f32": 4, "f64": 8}


def _transpose(name, dtype, size, perm, alpha=1.0, beta=0.0, outer_a="", outer_b=""):
    case = {"kind": "transpose", "dtype": dtype, "size": "x".join(map(str, size)),
            "perm": ",".join(map(str, perm)), "alpha": float(alpha), "beta": float(beta),
            "outer_a": outer_a, "outer_b": outer_b}
    return dict(case, name=name) if name else case


def _contract(name, dtype, spec, extents, alpha=1.0, beta=0.0):
    case = {"kind": "contract", "dtype": dtype, "spec": spec,
            "extents": ",".join(f"{m}{n}" for m, n in extents), "alpha": float(alpha),
            "beta": float(beta)}
    return dict(case, name=name) if name else case


def listed():
    sweep = {(w.size_a, w.perm): w for w in sweep57()}

    def swept(name, size, perm, beta):
        assert (size, perm) in sweep
        return _transpose(name, "f32", size, perm, 1.0, beta)

    gemm_c = CONTRACTIONS_BY_NAME["abcd_aebf_dfce"]
    gemm_a = CONTRACTIONS_BY_NAME["abcde_efbad_cf"]
    return [
        # the smallest: a cache-resident 3-D tensor, where the call and the launch count
        _transpose("small3d_f32", "f32", (48, 40, 32), (2, 0, 1)),
        # an ordinary 10 MB block of a larger array, odd extents, updated in place (a
        # tensor code's sub-block: outer sizes, fp64, alpha and beta)
        _transpose("block4d_f64_sub", "f64", (65, 33, 64, 9), (2, 0, 3, 1), 1.5, -0.5,
                   outer_a="72x33x65x9", outer_b="64x65x11x33"),
        # channels-last to channels-first: a batch of 64 x 3136 matrices, 51 MB
        _transpose("batched3d_f32", "f32", (64, 3136, 64), (1, 0, 2)),
        # matrix transposition, power-of-two extents
        _transpose("matrix8192_f32", "f32", (8192, 8192), (1, 0)),
        # matrix transposition, odd rows
        swept("matrix2193x22800_f32", (2193, 22800), (1, 0), 0.0),
        # index reversal of a ragged 4-D tensor, B updated
        swept("ragged4d_f32_beta1", (427, 110, 3, 355), (3, 2, 1, 0), 1.0),
        # stride-1 index kept, rows of odd length
        swept("keep4d_row75_f32", (75, 100, 11, 606), (0, 3, 2, 1), 0.0),
        # stride-1 index kept, fp64, B updated
        _transpose("keep4d_f64_beta", "f64", (96, 96, 96, 96), (0, 3, 2, 1), 2.0, 0.5),
        # 6-D, no extent a whole cache line, scaled
        _transpose("scaled6d_f32", "f32", (24, 20, 16, 24, 18, 20), (5, 2, 0, 4, 1, 3), 1.5),
        # the largest: 5-D with tiny leading extents, 708 MB, B updated
        _transpose("large5d_f32_beta1", "f32", (3, 2, 640, 480, 96), (4, 2, 0, 3, 1), 1.0, 1.0),
        # contraction with a large result and few contracted elements
        _contract("contract_abcd_aebf_dfce", gemm_c.dtype, gemm_c.spec, gemm_c.extents),
        # contraction whose operand and result are both reordered
        _contract("contract_abcde_efbad_cf", gemm_a.dtype, gemm_a.spec, gemm_a.extents),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _draw_transpose(rng):
    dtype = rng.choice(("f32", "f32", "f64"))
    alpha, beta = rng.choice(((1.0, 0.0), (1.0, 0.0), (1.5, 0.0), (1.0, 1.0), (2.0, 0.5)))
    moved = _log_uniform(rng, 4e5, 1.0e9)  # bytes an ideal implementation moves
    target = moved / ELEM[dtype] / (2 if beta == 0 else 3)
    while True:
        n = rng.randint(2, 6)
        shares = [rng.expovariate(1.0) for _ in range(n)]
        size = [max(2, round(target ** (s / sum(shares)))) for s in shares]
        size[-1] = max(2, round(target / math.prod(size[:-1])))
        perm = rng.sample(range(n), n)
        if 0.9 < math.prod(size) / target < 1.03 and perm != sorted(perm):
            break
    outer_a = outer_b = ""
    if rng.random() < 0.2:  # a block of larger tensors
        outer_a = "x".join(str(s + rng.randint(0, 8)) for s in size[:-1]) + f"x{size[-1]}"
        outer_b = "x".join(str(size[p] + rng.randint(0, 8)) for p in perm[:-1]) + f"x{size[perm[-1]]}"
        if _numel(outer_a) > 4 * math.prod(size) or _numel(outer_b) > 4 * math.prod(size):
            outer_a = outer_b = ""
    return _transpose("", dtype, size, perm, alpha, beta, outer_a, outer_b)


def _draw_contract(rng):
    dtype = rng.choice(("f32", "f64", "f64"))
    while True:
        m, n = _log_uniform(rng, 24, 1e4), _log_uniform(rng, 24, 1e4)
        k = _log_uniform(rng, 4, 1000)
        if (2 * m * n * k < 4e9 and (m * n + m * k + n * k) * ELEM[dtype] < 2.6e8
                and m * n * k > 1e6):
            break
    groups, letters = [], iter("abcdefgh")
    extents = []
    for v in (m, n, k):
        parts = 1 if v < 8 or rng.random() < 0.3 else 2
        first = round(_log_uniform(rng, 2, v / 2)) if parts == 2 else round(v)
        sizes = [first] + ([max(2, round(v / first))] if parts == 2 else [])
        names = [next(letters) for _ in sizes]
        extents += list(zip(names, sizes))
        groups.append(names)
    a, b, c = (rng.sample(x, len(x)) for x in (groups[0] + groups[2], groups[1] + groups[2],
                                                groups[0] + groups[1]))
    beta = rng.choice((0.0, 0.0, 1.0))
    return _contract("", dtype, f"{''.join(c)}={''.join(a)}*{''.join(b)}", extents, 1.0, beta)


def draw(rng):
    return _draw_contract(rng) if rng.random() < 0.2 else _draw_transpose(rng)


# ---------------------------------------------------------------------------
# What a case's texts say
# ---------------------------------------------------------------------------


def _ints(text, sep="x"):
    return tuple(int(x) for x in text.split(sep))


def _numel(text):
    return math.prod(_ints(text))


def _spec(case):
    """(modes_c, modes_a, modes_b, extent of each mode)"""
    c, ab = case["spec"].split("=")
    a, b = ab.split("*")
    return c, a, b, {x[0]: int(x[1:]) for x in case["extents"].split(",")}


def _uniform(n, dtype, seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 4 + stream)
    return torch.rand(n, dtype=TORCH[dtype], device="cuda", generator=g) * 2 - 1


def _inputs(case, seed):
    """Flat device tensors: the inputs and the tensor to be written or updated."""
    if case["kind"] == "contract":
        c, a, b, ext = _spec(case)
        na, nb, nc = (math.prod(ext[m] for m in x) for x in (a, b, c))
        return (_uniform(na, case["dtype"], seed, 0), _uniform(nb, case["dtype"], seed, 1),
                _uniform(nc, case["dtype"], seed, 2))
    na = _numel(case["outer_a"] or case["size"])
    nb = _numel(case["outer_b"] or case["size"])
    return _uniform(na, case["dtype"], seed, 0), _uniform(nb, case["dtype"], seed, 1)


def prepare(case, seed):
    if case["kind"] == "contract":
        c, a, b, ext = _spec(case)
        A, B, C = _inputs(case, seed)
        plan = contraction.Contraction(c, a, [ext[m] for m in a], b, [ext[m] for m in b],
                                       case["alpha"], case["beta"], case["dtype"])
        plan.workspace()  # allocated once, kept with the plan
        return {"plan": plan, "args": (A, B, C), "out": C}
    A, B = _inputs(case, seed)
    outer = {f"outer_size_{t}": _ints(case["outer_" + t]) for t in "ab" if case["outer_" + t]}
    plan = hptt.create_plan(_ints(case["perm"], ","), _ints(case["size"]), case["alpha"],
                            case["beta"], case["dtype"], **outer)
    return {"plan": plan, "args": (A, B), "out": B}


def run(state):
    state["plan"].exec(*state["args"])
    return state["out"]


def work(case):
    e = ELEM[case["dtype"]]
    updated = 1 if case["beta"] != 0 else 0
    if case["kind"] == "contract":
        c, a, b, ext = _spec(case)
        na, nb, nc = (math.prod(ext[m] for m in x) for x in (a, b, c))
        return {"bytes": e * (na + nb + nc * (1 + updated)), "flops": 2 * math.prod(ext.values())}
    n = _numel(case["size"])
    flops = n * (3 if updated else 0 if case["alpha"] == 1.0 else 1)
    return {"bytes": e * n * (2 + updated), "flops": flops}


def tolerance(case):
    if case["kind"] == "transpose":
        return "exact"  # one rounding each of alpha*a, beta*b and their sum
    # dot products of length k in another order: the rounding errors of k
    # additions add up like a random walk; measured against 64-bit torch on
    # the listed cases 1.7e-16 (k = 16 and 32), about 0.4 u sqrt(k), which
    # two orders may both be off, times about four
    c, a, b, ext = _spec(case)
    k = math.prod(ext[m] for m in a if m not in c)
    u = 2.0 ** -24 if case["dtype"] == "f32" else 2.0 ** -53
    return {"rel": 2 * u * math.sqrt(k), "max": min(0.5, 8 * u * math.sqrt(k))}


def _strided(flat, size, outer):
    """The block `size` of a flat Fortran-ordered tensor of extents `outer`
    (its first element first), as a view whose axes are in reverse order."""
    outer = outer or size
    strides, s = [], 1
    for x in outer:
        strides.append(s)
        s *= x
    return flat.as_strided(tuple(reversed(size)), tuple(reversed(strides)))


def exact(case, seed):
    alpha, beta = case["alpha"], case["beta"]
    if case["kind"] == "contract":
        c, a, b, ext = _spec(case)
        A, B, C = (t.double() for t in _inputs(case, seed))
        A = A.view([ext[m] for m in reversed(a)])
        B = B.view([ext[m] for m in reversed(b)])
        P = torch.einsum(f"{a[::-1]},{b[::-1]}->{c[::-1]}", A, B).reshape(-1)
        return alpha * P + (beta * C if beta != 0 else 0)
    size, perm = _ints(case["size"]), _ints(case["perm"], ",")
    A, B = (t.double() for t in _inputs(case, seed))
    n = len(size)
    src = _strided(A, size, _ints(case["outer_a"]) if case["outer_a"] else None)
    # axis j of a reversed view is index n-1-j
    src = src.permute([n - 1 - perm[n - 1 - j] for j in range(n)])
    dst = _strided(B, [size[p] for p in perm], _ints(case["outer_b"]) if case["outer_b"] else None)
    dst.copy_(alpha * src + (beta * dst if beta != 0 else 0))
    return B
