"""The products that this library's users have it do, as cases that can be timed and compared.

A case is one call of a public entry point on operands resident in HBM: `matmul` (which marshals to
oz2_ctx_dgemm / oz2_ctx_sgemm) or, for operands converted once, `oz2_dgemm_prepared` /
`oz2_sgemm_prepared`.  Its keys:

  dtype          "f64" (DGEMM) or "f32" (SGEMM)
  m, n, k        C is m x n, the contraction has k terms
  moduli         number of moduli: 14 to 18 match or exceed FP64, 6 to 9 FP32
  a_t, b_t       the operand is stored transposed (`X.t()` is passed)
  update         alpha = -1, beta = 1 (C <- C - A B, in place) instead of C <- A B
  accurate       accurate mode of the scale vectors
  prepared       both factors converted beforehand (oz2_prepare_*); the pass is the product only
  phi            spread of the entries (U - 0.5) exp(phi Z): 0.5 resembles dense linear algebra
"""
from __future__ import annotations

import math

import torch

import paper_2508_03984_amd as oz


def _case(name, dtype, m, n, k, moduli, *, a_t=False, b_t=False, update=False, accurate=False, prepared=False, phi=0.5):
    c = dict(dtype=dtype, m=m, n=n, k=k, moduli=moduli, a_t=a_t, b_t=b_t, update=update, accurate=accurate,
             prepared=prepared, phi=phi)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call of the benchmark's configurations: one block of a blocked algorithm, where latency counts
        _case("d_256", "f64", 256, 256, 256, 14),
        # a small single-precision product of no round size, e.g. a layer of a small network; B stored transposed
        _case("s_500x300x777", "f32", 500, 300, 777, 8, b_t=True),
        # a medium square product, where the native routine and the emulation cross over
        _case("d_1024", "f64", 1024, 1024, 1024, 15),
        # normal equations A^T B of two tall matrices with odd sizes, subtracted from C
        _case("d_1500x1111x3001_tn", "f64", 1500, 1111, 3001, 16, a_t=True, update=True, phi=1.0),
        # single precision in the middle of the range
        _case("s_2048", "f32", 2048, 2048, 2048, 7),
        # accurate mode, whose scale vectors need a product of their own
        _case("d_2048_accurate", "f64", 2048, 2048, 2048, 15, accurate=True),
        # the moduli count that is on par with native FP64, at the benchmark's middle size
        _case("d_4096", "f64", 4096, 4096, 4096, 14),
        # trailing update of a blocked LU factorisation
        _case("d_8192x8192x512_update", "f64", 8192, 8192, 512, 15, update=True),
        # two matrices that a program keeps converted and multiplies again and again
        _case("d_4096x3072x2048_prepared", "f64", 4096, 3072, 2048, 15, prepared=True),
        # a long contraction: inner products over many samples, wider exponent range
        _case("d_1536x1000x40000", "f64", 1536, 1000, 40000, 18, phi=1.0),
        # single precision at the benchmark's size
        _case("s_8192", "f32", 8192, 8192, 8192, 8),
        # the headline configuration
        _case("d_16384", "f64", 16384, 16384, 16384, 16),
    ]


_MAX_OPS = 2.0 * 16384.0**3 * 16


def _log_uniform(rng, lo, hi):
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    # round sizes are common in practice: multiples of 256 or 64 next to sizes of any kind
    to = rng.choice((1, 1, 1, 64, 256))
    return max(lo, min(hi, (v + to // 2) // to * to))


def draw(rng):
    while True:
        f64 = rng.random() < 0.65
        shape = rng.choice(("square", "any", "any", "short", "long"))
        if shape == "square":
            m = n = k = _log_uniform(rng, 200, 12000)
        elif shape == "any":
            m, n, k = (_log_uniform(rng, 100, 9000) for _ in range(3))
        elif shape == "short":      # rank-k updates
            m, n, k = _log_uniform(rng, 1500, 14000), _log_uniform(rng, 1500, 14000), _log_uniform(rng, 64, 1024)
        else:                       # long contractions
            m, n, k = _log_uniform(rng, 200, 2500), _log_uniform(rng, 200, 2500), _log_uniform(rng, 12000, 90000)
        moduli = rng.randint(14, 18) if f64 else rng.randint(6, 9)
        if 2.0 * m * n * k * moduli > 0.5 * _MAX_OPS:
            continue
        prepared = rng.random() < 0.15
        return _case(None, "f64" if f64 else "f32", m, n, k, moduli, a_t=rng.random() < 0.3, b_t=rng.random() < 0.4,
                     update=shape == "short" or rng.random() < 0.2, accurate=not prepared and rng.random() < 0.2,
                     prepared=prepared, phi=rng.choice((0.5, 0.5, 1.0)))


def _inputs(case, seed):
    """A, B as the caller holds them (a transposed view where the case says so), and C before the call."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    dtype = torch.float64 if case["dtype"] == "f64" else torch.float32

    def matrix(rows, cols):
        out = torch.empty((rows, cols), dtype=dtype, device="cuda")
        step = max(1, (1 << 26) // cols)                 # temporaries of a block of rows only
        for r in range(0, rows, step):
            shape = (min(step, rows - r), cols)
            u = torch.rand(shape, dtype=torch.float64, device="cuda", generator=gen)
            z = torch.randn(shape, dtype=torch.float64, device="cuda", generator=gen)
            out[r:r + step] = ((0.5 - u) * torch.exp(case["phi"] * z)).to(dtype)
        return out

    m, n, k = case["m"], case["n"], case["k"]
    A = matrix(k, m).t() if case["a_t"] else matrix(m, k)
    B = matrix(n, k).t() if case["b_t"] else matrix(k, n)
    C = matrix(m, n) if case["update"] else torch.empty((m, n), dtype=dtype, device="cuda")
    return A, B, C


def prepare(case, seed):
    A, B, C = _inputs(case, seed)
    state = dict(case=case, A=A, B=B, C=C)
    if case["prepared"]:
        convert = oz.oz2_prepare_d if case["dtype"] == "f64" else oz.oz2_prepare_s
        op_a, ld_a = (oz.OZ2_OP_T, case["m"]) if case["a_t"] else (oz.OZ2_OP_N, case["k"])
        op_b, ld_b = (oz.OZ2_OP_T, case["k"]) if case["b_t"] else (oz.OZ2_OP_N, case["n"])
        state["left"] = convert(0, op_a, case["m"], case["k"], A, ld_a, case["moduli"])
        state["right"] = convert(1, op_b, case["n"], case["k"], B, ld_b, case["moduli"])
        torch.cuda.synchronize()
    return state


def run(state):
    case, C = state["case"], state["C"]
    alpha, beta = (-1.0, 1.0) if case["update"] else (1.0, 0.0)
    if case["prepared"]:
        product = oz.oz2_dgemm_prepared if case["dtype"] == "f64" else oz.oz2_sgemm_prepared
        product(state["left"], state["right"], alpha, beta, C, case["n"])
        return C
    return oz.matmul(state["A"], state["B"], case["moduli"], alpha=alpha, beta=beta, out=C, accurate=case["accurate"])


def work(case):
    """Inputs read once (the prepared form: their residues), C written once (an update reads it too), and
    the INT8 products of the scheme: one multiply-add per modulus and term, one more product in accurate mode."""
    m, n, k, moduli = case["m"], case["n"], case["k"], case["moduli"]
    e = 8 if case["dtype"] == "f64" else 4
    operand = moduli if case["prepared"] else e
    return {"bytes": float(operand * (m * k + k * n) + e * m * n * (2 if case["update"] else 1)),
            "flops": 2.0 * m * n * k * (moduli + (1 if case["accurate"] else 0))}


def tolerance(case):
    """What the truncation to the moduli's range leaves (it shrinks by about 2^-4 per modulus), or the
    output type's rounding and, in FP64, that of the product compared with.  Measured against `exact`:
    FP64 9.5e-15 at 14 moduli (k = 4096), 1e-15 to 7e-15 (k = 256 to 40000) from 15 on; FP32 2.4e-6 at 6
    (k = 1000), 5.7e-7 at 7 (k = 2048), 4.5e-8 at 8 (k = 8192).  About four times these."""
    if case["dtype"] == "f64":
        return {"rel": max(2e-14, 5e-14 * 16.0 ** (14 - case["moduli"]))}
    return {"rel": max(1e-7, 4e-5 * 16.0 ** (6 - case["moduli"]))}


def exact(case, seed):
    A, B, C = _inputs(case, seed)
    AB = torch.matmul(A.double().contiguous(), B.double().contiguous())
    return C.double() - AB if case["update"] else AB
