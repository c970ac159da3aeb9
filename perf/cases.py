"""Performance cases of the FP64 product emulated with INT8 products: what its callers do, over the range they do it in.

A case is one call of an entry point on column-major FP64 matrices that are resident in device memory, with a
context (settings and workspace) that the program keeps:
  entry "dgemm"   C := alpha op(A) op(B) + beta C
        "static"  C := A B on the library's own static workspace (callers that cannot allocate)
        "dsyrk"   one triangle of C := alpha op(A) op(A)^T + beta C
        "dtrmm"   X := alpha op(A) X or alpha X op(A), A triangular; the program keeps X's input, so a pass copies it first
  m, n, k, moduli; phi: spread of the inputs (rand - 0.5) exp(phi randn); mode: shift selection (0 maxima, 1
  Cauchy-Schwarz, 2 INT8-product bound); ta, tb, alpha, beta, uplo, side, diag as in the BLAS.
For dsyrk m == n is the order of C; for dtrmm X is m x n and k the order of A (m on the left, n on the right).
"""
import math

import torch

import paper_2504_08009_amd as oz

DEVICE = "cuda:0"
FULL = dict(entry="dgemm", phi=0.5, mode=0, ta="N", tb="N", alpha=1.0, beta=0.0, uplo="L", side="L", diag="N")


def _case(name, m, n, k, moduli, **more):
    return dict(FULL, name=name, m=m, n=n, k=k, moduli=moduli, **more)


def listed():
    return [
        # the smallest products, made many times in a row by code that cannot allocate: latency and launches decide
        _case("static_256", 256, 256, 256, 14, entry="static"),
        # small blocks of a blocked factorisation: odd sizes, a transposed operand, an update of C
        _case("update_333x517x291_tn", 333, 517, 291, 15, ta="T", alpha=-1.0, beta=1.0),
        # the ordinary small product with FP64-level accuracy
        _case("square_1024", 1024, 1024, 1024, 14),
        # the smallest size of the published tables, with the Cauchy-Schwarz ("fast") shifts they time
        _case("square_2048_fast", 2048, 2048, 2048, 14, mode=1),
        # many right-hand sides: a large matrix against a few vectors, reading it is most of the work
        _case("block_of_vectors_8192x96", 8192, 96, 8192, 16),
        # a medium product of ragged sizes with the INT8-product ("accurate") shifts, second operand transposed
        _case("ragged_3001x2777x3500_nt_accurate", 3001, 2777, 3500, 15, mode=2, tb="T", phi=1.0),
        # the benchmark's medium square product
        _case("square_4096", 4096, 4096, 4096, 16, phi=1.0),
        # symmetric update of a Cholesky factorisation: a panel against itself, lower triangle
        _case("dsyrk_5000x1024", 5000, 5000, 1024, 16, entry="dsyrk", alpha=-1.0, beta=1.0),
        # triangular product in place, as a blocked inversion makes them
        _case("dtrmm_4096x2048", 4096, 2048, 4096, 16, entry="dtrmm"),
        # an outer-product-like update: a large C from a short inner dimension, wide spread of the inputs
        _case("outer_8192x8192x1024", 8192, 8192, 1024, 18, phi=4.0),
        # the headline product
        _case("square_16384", 16384, 16384, 16384, 16),
        # the longest inner dimension of the benchmark
        _case("long_8192x8192x65536", 8192, 8192, 65536, 18, phi=4.0),
    ]


MOST_WORK = 2.0 * 16384 ** 3 * 16


def draw(rng):
    def size(low, high):
        v = int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))
        return v if rng.random() < 0.7 else max(64, v // 64 * 64)

    while True:
        c = dict(FULL, moduli=rng.randint(10, 18), phi=rng.choice([0.5, 1.0, 2.0, 4.0]))
        c["entry"] = rng.choice(["dgemm"] * 7 + ["static", "dsyrk", "dtrmm"])
        c["m"], c["n"], c["k"] = size(64, 16384), size(64, 16384), size(64, 32768)
        if c["entry"] == "static":
            c["m"], c["n"], c["k"] = size(64, 1024), size(64, 1024), size(64, 1024)
        elif c["entry"] == "dsyrk":
            c["n"] = c["m"]
            c.update(uplo=rng.choice("LU"), ta=rng.choice("NT"), alpha=rng.choice([1.0, -1.0]), beta=rng.choice([0.0, 1.0]))
        elif c["entry"] == "dtrmm":
            c.update(uplo=rng.choice("LU"), side=rng.choice("LR"), ta=rng.choice("NT"), diag=rng.choice("NU"))
            c["k"] = c["m"] if c["side"] == "L" else c["n"]
        else:
            c.update(ta=rng.choice("NNT"), tb=rng.choice("NNT"), mode=rng.choice([0, 0, 0, 1, 2]))
            if rng.random() < 0.4:
                c.update(alpha=-1.0, beta=1.0)
        if work(c)["flops"] <= MOST_WORK:
            return c


def _matrix(gen, rows, cols, phi):
    """rows x cols values in column-major order, as the (cols, rows) tensor whose memory that is"""
    x = torch.randn((cols, rows), dtype=torch.float64, device=DEVICE, generator=gen).mul_(phi).exp_()
    return x.mul_(torch.rand((cols, rows), dtype=torch.float64, device=DEVICE, generator=gen).sub_(0.5))


def _inputs(case, seed):
    m, n, k, phi = case["m"], case["n"], case["k"], case["phi"]
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    if case["entry"] == "dtrmm":
        return _matrix(gen, k, k, phi), None, _matrix(gen, m, n, phi)
    a = _matrix(gen, *((m, k) if case["ta"] == "N" else (k, m)), phi)
    b = None if case["entry"] == "dsyrk" else _matrix(gen, *((k, n) if case["tb"] == "N" else (n, k)), phi)
    if case["beta"]:
        return a, b, _matrix(gen, m, n, phi)
    # what a result that is only written holds before; the triangle that dsyrk does not write stays as it is
    return a, b, torch.zeros((n, m), dtype=torch.float64, device=DEVICE)


def prepare(case, seed):
    a, b, c = _inputs(case, seed)
    s = dict(case, a=a, b=b, c=c)
    if case["entry"] == "static":
        oz.oz2_init()
        return s
    ctx = oz.Context()
    ctx.set(oz.OZ2_OPT_SHIFT_MODE, case["mode"])
    ctx.allocate_workspace(case["m"], case["n"], case["k"], case["moduli"], device=DEVICE)
    s["ctx"] = ctx
    if case["entry"] == "dtrmm":
        s["x"] = torch.empty_like(c)
    return s


def run(s):
    m, n, k, a, b, c = s["m"], s["n"], s["k"], s["a"], s["b"], s["c"]
    if s["entry"] == "static":
        oz.oz2_dgemm_static(m, n, k, a.data_ptr(), m, b.data_ptr(), k, c.data_ptr(), m, s["moduli"])
        return c
    if s["entry"] == "dsyrk":
        s["ctx"].dsyrk(s["uplo"], s["ta"], n, k, s["alpha"], a.data_ptr(), a.shape[1], s["beta"], c.data_ptr(), m, s["moduli"])
        return c
    if s["entry"] == "dtrmm":
        x = s["x"].copy_(c)
        s["ctx"].dtrmm(s["side"], s["uplo"], s["ta"], s["diag"], m, n, s["alpha"], a.data_ptr(), k, x.data_ptr(), m, s["moduli"])
        return x
    s["ctx"].dgemm(s["ta"], s["tb"], m, n, k, s["alpha"], a.data_ptr(), a.shape[1], b.data_ptr(), b.shape[1], s["beta"],
                   c.data_ptr(), m, s["moduli"])
    return c


def work(case):
    """Bytes: each FP64 operand read once, the result written once (and read where it is updated).  Operations: one
    INT8 product per modulus, which the method is; half of it where half of the product is zero or not wanted."""
    m, n, k = case["m"], case["n"], case["k"]
    ops = 2.0 * m * n * k * case["moduli"]
    touched = 2 if case["beta"] or case["entry"] == "dtrmm" else 1
    if case["entry"] == "dsyrk":
        return {"bytes": 8.0 * (n * k + touched * n * (n + 1) / 2), "flops": ops / 2}
    if case["entry"] == "dtrmm":
        return {"bytes": 8.0 * (k * (k + 1) / 2 + touched * m * n), "flops": ops / 2}
    return {"bytes": 8.0 * (m * k + k * n + touched * m * n), "flops": ops}


def tolerance(case):
    """The method works in exact integers between one truncation of the inputs and one rounding of the result, and the
    library's results are the oracle's bit for bit: there is one right value for every element."""
    return "exact"


def exact(case, seed):
    """The same product by torch in FP64 (its own rounding errors are larger than those of 16 or more moduli)."""
    a, b, c = _inputs(case, seed)
    if case["entry"] == "dtrmm":
        t = torch.tril(a.t()) if case["uplo"] == "L" else torch.triu(a.t())
        if case["diag"] == "U":
            t.diagonal().fill_(1.0)
        t = t if case["ta"] == "N" else t.t()
        p = torch.matmul(t, c.t()) if case["side"] == "L" else torch.matmul(c.t(), t)
        return (case["alpha"] * p).t().contiguous()
    opa = a.t() if case["ta"] == "N" else a
    if case["entry"] == "dsyrk":
        opb = opa.t()
    else:
        opb = b.t() if case["tb"] == "N" else b
    p = torch.matmul(opa, opb).mul_(case["alpha"])
    if case["beta"]:
        p.add_(c.t(), alpha=case["beta"])
    if case["entry"] == "dsyrk":
        rows = torch.arange(case["n"], device=DEVICE)
        mine = rows[:, None] >= rows[None, :] if case["uplo"] == "L" else rows[:, None] <= rows[None, :]
        p = torch.where(mine, p, c.t())
    return p.t().contiguous()
