"""Performance cases of the library: what its users have it compute, through
the Python entry points, from the smallest orders to the largest.

Kinds
-----
* ``factor``     one dense skew-symmetric matrix: ``factor`` + ``pfaffian``
                 (float64; complex128 for a complex skew-symmetric matrix).
* ``pfaffian``   the Pfaffian alone, by the even column steps
                 (``pfaffian_direct``; float64 and float32).
* ``batched``    many small matrices at once (``factor_batched``).
* ``solve``      right-hand sides solved with factors the program keeps.
* ``conv``       one convolution layer (``convgemm``, float32).

The factorizations work in place, so a program that has matrices of its own
puts each one into the working buffer first: ``run`` does the same, and that
copy is part of its time (about 1 % of the large orders' time, a third of
the batched call's).

Inputs are drawn on the GPU from the seed: Gaussian skew-symmetric matrices
(``graded``: entries spread over six decades, the input on which the pivot
order matters most), activations uniform on [0, 1) and He-style Gaussian
filters for the convolutions, the distributions the repository's generators
and benchmark use.
"""
from __future__ import annotations

import math

import torch

import paper_2005_06410_amd as lt

_DTYPES = {"f64": torch.float64, "f32": torch.float32, "c128": torch.complex128}
_EXACT_ORDER = 6000   # largest order whose reduction exact() repeats step by step


def listed():
    return [
        # -- one matrix, factors and Pfaffian --------------------------------
        # smallest configured order: a call inside a loop over small systems,
        # where launches and the latency of a column step are everything
        {"name": "factor_256", "kind": "factor", "n": 256, "dtype": "f64", "graded": False},
        # ordinary order of the configurations
        {"name": "factor_2048", "kind": "factor", "n": 2048, "dtype": "f64", "graded": False},
        # the benchmark's order, the largest
        {"name": "factor_16384", "kind": "factor", "n": 16384, "dtype": "f64", "graded": False},
        # a complex matrix of ragged order (no multiple of any tile)
        {"name": "factor_1501_complex", "kind": "factor", "n": 1501, "dtype": "c128", "graded": False},
        # -- the Pfaffian alone ------------------------------------------------
        # single precision, graded entries, an order off every block size
        {"name": "pfaffian_5002_f32", "kind": "pfaffian", "n": 5002, "dtype": "f32", "graded": True},
        # -- many small matrices ------------------------------------------------
        # the configured batch: 8192 matrices of order 64
        {"name": "batched_8192x64", "kind": "batched", "n": 64, "batch": 8192, "dtype": "f64"},
        # smaller matrices in single precision, an order off every block size
        {"name": "batched_5000x22_f32", "kind": "batched", "n": 22, "batch": 5000, "dtype": "f32"},
        # -- solving with kept factors -------------------------------------------
        # one right-hand side at the benchmark's order: each new b costs this
        {"name": "solve_16384", "kind": "solve", "n": 16384, "nrhs": 1},
        # -- convolution layers -----------------------------------------------------
        # AlexNet's second convolution at the benchmarked batch: the largest GEMM
        {"name": "conv_alexnet4_b80", "kind": "conv", "kn": 192, "k": 5, "ci": 64, "h": 55, "w": 55, "b": 80,
         "stride": 1, "pad": 0},
        # its fourth one on a single image: inference latency, few output positions
        {"name": "conv_alexnet7_b1", "kind": "conv", "kn": 384, "k": 3, "ci": 384, "h": 13, "w": 13, "b": 1,
         "stride": 1, "pad": 0},
        # a "same" 3 x 3 layer (padding 1), the usual form of the later layers
        {"name": "conv_same3x3_b16", "kind": "conv", "kn": 384, "k": 3, "ci": 192, "h": 27, "w": 27, "b": 16,
         "stride": 1, "pad": 1},
        # AlexNet's first layer: three channels, 11 x 11 taps, stride 4
        {"name": "conv_alexnet2_b32", "kind": "conv", "kn": 64, "k": 11, "ci": 3, "h": 224, "w": 224, "b": 32,
         "stride": 4, "pad": 0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["factor", "factor", "pfaffian", "batched", "solve", "conv", "conv"])
    if kind == "factor":
        dtype = rng.choice(["f64", "f64", "c128"])
        n = _log_int(rng, 100, 9000 if dtype == "f64" else 3000)
        return {"kind": kind, "n": n, "dtype": dtype, "graded": False}
    if kind == "pfaffian":
        dtype = rng.choice(["f64", "f32"])
        return {"kind": kind, "n": 2 * _log_int(rng, 50, 4500), "dtype": dtype, "graded": dtype == "f32"}
    if kind == "batched":
        dtype = rng.choice(["f64", "f32"])
        n = rng.randint(6, 64) if dtype == "f64" else 2 * rng.randint(3, 32)   # an odd order's Pfaffian is 0
        return {"kind": kind, "n": n, "batch": _log_int(rng, 100, 30000), "dtype": dtype}
    if kind == "solve":
        return {"kind": kind, "n": 2 * _log_int(rng, 100, 6000), "nrhs": rng.choice([1, 1, 2, 5, 8, 16])}
    while True:
        k = rng.choice([1, 3, 3, 5, 7])
        c = {"kind": kind, "kn": _log_int(rng, 16, 512), "k": k, "ci": rng.choice([3, 16, 33, 64, 128, 192, 256, 384]),
             "h": rng.randint(7, 64), "w": rng.randint(7, 64), "b": _log_int(rng, 1, 64),
             "stride": rng.choice([1, 1, 1, 2]), "pad": rng.choice([0, k // 2])}
        if 1e6 < work(c)["flops"] < 1e11:
            return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _skew(n, dtype, graded, seed, batch=None):
    """Column-major skew-symmetric matrix (or a batch of them), entries drawn
    for the strict lower triangle.  Row-major Y = -X^T reads column-major as X."""
    g = _gen(seed)
    shape = (n, n) if batch is None else (batch, n, n)
    if dtype == "c128":
        T = torch.complex(torch.randn(shape, generator=g, device="cuda", dtype=torch.float64),
                          torch.randn(shape, generator=g, device="cuda", dtype=torch.float64))
    else:
        T = torch.randn(shape, generator=g, device="cuda", dtype=torch.float64)
        if graded:
            T *= torch.pow(10.0, 6.0 * torch.rand(shape, generator=g, device="cuda", dtype=torch.float64) - 3.0)
        T = T.to(_DTYPES[dtype])
    T.triu_(1)
    Y = T - T.mT
    return Y.mT               # stride(0) == 1 in each matrix


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("factor", "pfaffian"):
        X = _skew(case["n"], case["dtype"], case["graded"], seed)
        return {"case": case, "X": X, "A": torch.empty_like(X),
                "ipiv": torch.empty(case["n"], dtype=torch.int32, device="cuda")}
    if kind == "batched":
        X = _skew(case["n"], case["dtype"], False, seed, case["batch"])
        return {"case": case, "X": X, "A": torch.empty_like(X),
                "ipiv": torch.empty((case["batch"], case["n"]), dtype=torch.int32, device="cuda")}
    if kind == "solve":
        n, nrhs = case["n"], case["nrhs"]
        A = _skew(n, "f64", False, seed)
        ipiv = lt.factor(A, check=True)
        b = torch.randn((nrhs, n), generator=_gen(seed + 7919), device="cuda", dtype=torch.float64)
        return {"case": case, "A": A, "ipiv": ipiv, "b": b.t(), "x": torch.empty_like(b).t()}
    g = _gen(seed)
    k, ci, kn = case["k"], case["ci"], case["kn"]
    # leftmost index fastest: a contiguous tensor with the axes reversed
    I = torch.rand((case["b"], ci, case["w"], case["h"]), generator=g, device="cuda")
    F = torch.randn((ci, k, k, kn), generator=g, device="cuda") * math.sqrt(2.0 / (k * k * ci))
    return {"case": case, "F": F.permute(3, 2, 1, 0), "I": I.permute(3, 2, 1, 0)}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "factor":
        A = state["A"].copy_(state["X"])
        ipiv = lt.factor(A, state["ipiv"])
        logabs, sign = lt.pfaffian(A, ipiv)
        return {"A": A, "ipiv": ipiv, "logabs": logabs, "sign": sign}
    if kind == "pfaffian":
        A = state["A"].copy_(state["X"])
        _, logabs, sign = lt.pfaffian_direct(A, ipiv=state["ipiv"])
        return {"logabs": logabs, "sign": sign}
    if kind == "batched":
        A = state["A"].copy_(state["X"])
        ipiv, logabs, sign = lt.factor_batched(A, state["ipiv"])
        if case["dtype"] == "f32":
            # two float32 pivots of almost the same size may be taken either
            # way, and the factors then differ altogether; the Pfaffian does not
            return {"logabs": logabs, "sign": sign}
        return {"A": A, "ipiv": ipiv, "logabs": logabs, "sign": sign}
    if kind == "solve":
        x = state["x"].copy_(state["b"])
        return lt.solve(state["A"], state["ipiv"], x)
    return lt.convgemm(state["F"], state["I"], stride=case["stride"], pad=case["pad"])


# ---------------------------------------------------------------------------
# what a pass cannot do without, and how exact it is
# ---------------------------------------------------------------------------
def _out(case):
    return tuple((case[d] - case["k"] + 2 * case["pad"]) // case["stride"] + 1 for d in ("h", "w"))


def work(case):
    kind = case["kind"]
    if kind == "conv":
        ho, wo = _out(case)
        kk, npos = case["k"] * case["k"] * case["ci"], ho * wo * case["b"]
        return {"bytes": 4.0 * (case["kn"] * kk + case["h"] * case["w"] * case["ci"] * case["b"] + case["kn"] * npos),
                "flops": 2.0 * case["kn"] * kk * npos}
    n = case["n"]
    tri = n * (n - 1) / 2.0
    if kind == "solve":
        return {"bytes": 8.0 * (tri + 2 * n * case["nrhs"]) + 4 * n, "flops": 2.0 * n * n * case["nrhs"]}
    elem = {"f64": 8, "f32": 4, "c128": 16}[case["dtype"]]
    flops = n ** 3 / 3.0 * (4 if case["dtype"] == "c128" else 1)
    if kind == "pfaffian":   # the matrix is workspace: read, not returned
        return {"bytes": float(elem * tri + 4 * n), "flops": flops}
    batch = case.get("batch", 1)
    return {"bytes": float(batch * (2 * elem * tri + 4 * n)), "flops": flops * batch}


def tolerance(case):
    """About four times the distance measured from the 64-bit results (over
    several seeds and orders), with room for unlucky condition numbers where
    both sides' errors grow with them."""
    kind = case["kind"]
    if kind == "conv":        # float32 sums of up to 10^4 terms in any order: 7e-7
        return {"rel": 3e-6, "max": 5e-5}
    if kind == "solve":       # 1e-11 at n = 3000 to 5000, growing with the order
        return {"rel": 1e-9, "max": 1e-8}
    if case["dtype"] == "f32":
        if kind == "batched":   # 1e-5 over the batch, 1e-3 for one nearly singular member
            return {"rel": 4e-5, "max": 1e-2, "differ": 0.001}
        return {"rel": 1e-6, "max": 1e-6}
    # factors 5e-14 at n = 3000, growing with the order; the complex phase 1e-12
    return {"rel": 1e-11, "max": 1e-9}


# ---------------------------------------------------------------------------
# the same results in 64 bits, with torch alone
# ---------------------------------------------------------------------------
def _reduce(X):
    """P X P^T = L T L^T step by step on a batch (B, n, n): the packed lower
    triangle (alpha_k at (k+1, k), L(r, k+1) at (r, k)), ipiv, alphas."""
    A = X.clone(memory_format=torch.contiguous_format)
    B, n, _ = A.shape
    ar = torch.arange(B, device=A.device)
    ipiv = torch.arange(n, device=A.device).repeat(B, 1)
    for k in range(n - 1):
        col = A[:, k + 1:, k]
        mag = (col.real.abs() + col.imag.abs()) if A.is_complex() else col.abs()
        p = mag.argmax(1) + k + 1
        ipiv[:, k + 1] = p
        pair = torch.stack([torch.full_like(p, k + 1), p], 1)
        i0, i1 = ar[:, None], pair
        A[i0, i1.flip(1)] = A[i0, i1]                        # rows k+1 and p
        at = A.transpose(1, 2)
        at[i0, i1.flip(1)] = at[i0, i1]                      # columns k+1 and p
        if k + 2 < n:
            alpha = A[:, k + 1, k].clone()
            l = torch.where((alpha != 0)[:, None], A[:, k + 2:, k] / alpha[:, None], torch.zeros_like(A[:, k + 2:, k]))
            v = A[:, k + 2:, k + 1].clone()
            U, V = torch.stack([l, -v], 2), torch.stack([v, l], 1)
            A[:, k + 2:, k + 2:] += torch.matmul(U, V) if B == 1 else U[:, :, :1] * V[:, :1] + U[:, :, 1:] * V[:, 1:]
            A[:, k + 2:, k] = l
    return A, ipiv.to(torch.int32)


def _pfaffian_of(A, ipiv):
    B, n, _ = A.shape
    ar = torch.arange(n, device=A.device)
    odd = (ipiv != ar).sum(1) % 2
    if n % 2:
        logabs = torch.full((B,), -math.inf, dtype=torch.float64, device=A.device)
        sign = torch.zeros(B, dtype=torch.complex128 if A.is_complex() else torch.int32, device=A.device)
        return logabs, sign
    a = -torch.diagonal(A, -1, 1, 2)[:, ::2]
    logabs = a.abs().log().sum(1)
    sign = torch.prod(a / a.abs(), 1) * torch.where(odd == 1, -1.0, 1.0)
    return logabs, sign if A.is_complex() else sign.round().to(torch.int32)


def exact(case, seed):
    kind = case["kind"]
    if kind == "conv":
        s = prepare(case, seed)
        ho, wo = _out(case)
        W = s["F"].permute(0, 3, 2, 1).double().reshape(case["kn"], -1)
        I = s["I"].permute(3, 2, 1, 0)
        O = torch.empty((case["b"], case["kn"], wo * ho), dtype=torch.float64, device="cuda")
        for i in range(case["b"]):
            cols = torch.nn.functional.unfold(I[i:i + 1].double(), case["k"], padding=case["pad"], stride=case["stride"])
            O[i] = W @ cols[0]
        return O.reshape(case["b"], case["kn"], wo, ho).permute(1, 3, 2, 0)
    n = case["n"]
    if kind == "solve":
        if n > _EXACT_ORDER:
            return None
        b = torch.randn((case["nrhs"], n), generator=_gen(seed + 7919), device="cuda", dtype=torch.float64)
        return torch.linalg.solve(_skew(n, "f64", False, seed).contiguous(), b.t().contiguous())
    if n > _EXACT_ORDER:
        return None
    X = _skew(n, case["dtype"], case.get("graded", False), seed, case.get("batch"))
    X64 = X if X.is_complex() else X.double()
    A, ipiv = _reduce(X64 if kind == "batched" else X64[None])
    logabs, sign = _pfaffian_of(A, ipiv)
    if kind == "pfaffian" or case["dtype"] == "f32":
        return {"logabs": logabs, "sign": sign}
    A = torch.tril(A, -1) + torch.triu(X64)                  # the upper triangle is never written
    if kind == "batched":
        return {"A": A, "ipiv": ipiv, "logabs": logabs, "sign": sign}
    return {"A": A[0], "ipiv": ipiv[0], "logabs": logabs, "sign": sign}
