"""Timed workloads of the library: what a program that uses it has it do.

Every case goes through a public entry point of the binding: `moa_gemm` with a
prepared descriptor (a program that repeats a product keeps its descriptor),
`moa_gemm_grouped` and `moa_gemm_batched` for many products at once, and the
two elementwise members of the ipophp family. Sizes are those of the benchmark
and its sweeps (256^3 FP64, 8192^3 FP32, 8192 x 4096 x 8192 scaled, 512
log-uniform products, the serving mix, long-k products, 64^2 (x) 128^2) and
ragged ones of the same ranges.

A case is a dict of plain values:
  kind "gemm":  m, n, p, dtype, path, one_term, accumulate, a_col, b_col
  kind "group": count, mp_lo, mp_hi, n_lo, n_hi, fp8_percent, shape_seed
  kind "batched": batch, m, n, p
  kind "kronecker": m, n, p, q, dtype      kind "hadamard": m, n, dtype
"""
from __future__ import annotations

import math
import random

import torch

from paper_2306_11148_amd import moa

DTYPES = {"f64": torch.float64, "f32": torch.float32}
SIZES = {"f64": 8, "f32": 4}


def _gemm(name, m, n, p, path="auto", dtype="f32", one_term=False, accumulate=False, a_col=False, b_col=False):
    c = {"kind": "gemm", "m": m, "n": n, "p": p, "dtype": dtype, "path": path, "one_term": one_term,
         "accumulate": accumulate, "a_col": a_col, "b_col": b_col}
    return c if name is None else {"name": name, **c}


def _group(name, count, mp_lo, mp_hi, n_lo, n_hi, fp8_percent, shape_seed):
    c = {"kind": "group", "count": count, "mp_lo": mp_lo, "mp_hi": mp_hi, "n_lo": n_lo, "n_hi": n_hi,
         "fp8_percent": fp8_percent, "shape_seed": shape_seed}
    return c if name is None else {"name": name, **c}


def listed():
    return [
        # the paper-sized FP64 product: launch and latency bound
        _gemm("f64_256", 256, 256, 256, dtype="f64"),
        # an FP64 update C += A B of a ragged shape, the paper's precision at an ordinary size
        _gemm("f64_ragged_update", 1999, 1531, 2113, dtype="f64", accumulate=True),
        # the plain ONF loop in FP32 at the benchmark's size (the kernel the headline is compared with)
        _gemm("onf_f32_8192", 8192, 8192, 8192, path="onf"),
        # the smallest default-path products: a small layer, one call at a time
        _gemm("split_192x320x160", 192, 320, 160),
        # a weight gradient X^T dY accumulated into a ragged matrix (X read column by column)
        _gemm("split_ragged_wgrad", 1531, 2029, 1237, accumulate=True, a_col=True),
        # the headline workload: square FP32 product on the default path
        _gemm("split_8192", 8192, 8192, 8192),
        # few blocks and a long k walk (Gram matrices, gradients over a long batch)
        _gemm("split_512x32768x512", 512, 32768, 512),
        # scaled FP8, two terms (the path's default), rows and columns of widely different scale
        _gemm("fp8_8192x4096x8192", 8192, 4096, 8192, path="fp8"),
        # scaled FP8, one term, ragged, against a weight stored row by output (B column-major)
        _gemm("fp8_one_term_ragged", 3001, 2777, 1999, path="fp8", one_term=True, b_col=True),
        # the batching workload: 512 independent products in one call
        _group("group_512", 512, 32, 2048, 32, 2048, 0, 4),
        # one admitted serving group: mixed shapes, 70% default path and 30% two-term FP8
        _group("group_serving", 32, 64, 4096, 64, 8192, 30, 5),
        # Kronecker product written once to memory
        {"name": "kronecker_8192", "kind": "kronecker", "m": 64, "n": 64, "p": 128, "q": 128, "dtype": "f32"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["f64", "f64", "onf", "mfma_f32", "split", "split", "split", "long_k", "fp8", "fp8", "group",
                       "serving", "batched", "kronecker", "hadamard"])
    acc = rng.random() < 0.3
    a_col, b_col = rng.random() < 0.25, rng.random() < 0.25
    if kind == "f64":
        return _gemm(None, _log(rng, 32, 4096), _log(rng, 32, 4096), _log(rng, 32, 4096), dtype="f64",
                     accumulate=acc, a_col=a_col, b_col=b_col)
    if kind in ("onf", "mfma_f32"):
        return _gemm(None, _log(rng, 64, 6144), _log(rng, 64, 6144), _log(rng, 64, 6144), path=kind, accumulate=acc,
                     a_col=a_col, b_col=b_col)
    if kind == "split":
        return _gemm(None, _log(rng, 32, 8192), _log(rng, 32, 8192), _log(rng, 32, 8192), accumulate=acc,
                     a_col=a_col, b_col=b_col)
    if kind == "long_k":
        return _gemm(None, _log(rng, 64, 1024), _log(rng, 4096, 65536), _log(rng, 64, 1024), accumulate=acc,
                     a_col=a_col)
    if kind == "fp8":
        return _gemm(None, _log(rng, 64, 8192), _log(rng, 64, 8192), _log(rng, 64, 8192), path="fp8",
                     one_term=rng.random() < 0.4, accumulate=acc, b_col=b_col)
    if kind == "group":
        return _group(None, _log(rng, 8, 512), 32, 2048, 32, 2048, 0, rng.randrange(1 << 20))
    if kind == "serving":
        return _group(None, _log(rng, 4, 64), 64, 2048, 64, 4096, 30, rng.randrange(1 << 20))
    if kind == "batched":
        return {"kind": "batched", "batch": _log(rng, 4, 128), "m": _log(rng, 32, 1024), "n": _log(rng, 32, 1024),
                "p": _log(rng, 32, 1024)}
    dtype = rng.choice(["f32", "f64"])
    if kind == "kronecker":
        return {"kind": "kronecker", "m": _log(rng, 4, 80), "n": _log(rng, 4, 80), "p": _log(rng, 16, 100),
                "q": _log(rng, 16, 100), "dtype": dtype}
    return {"kind": "hadamard", "m": _log(rng, 64, 8192), "n": _log(rng, 64, 8192), "dtype": dtype}


def _shapes(case):
    """(m, n, p, fp8) of every member of a group."""
    r = random.Random(case["shape_seed"])
    return [(_log(r, case["mp_lo"], case["mp_hi"]), _log(r, case["n_lo"], case["n_hi"]),
             _log(r, case["mp_lo"], case["mp_hi"]), r.randrange(100) < case["fp8_percent"])
            for _ in range(case["count"])]


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _draw_operands(case, seed):
    """A, B and C (the old C, or memory for the result) of a "gemm" case."""
    g = _generator(seed)
    dt, m, n, p = DTYPES[case["dtype"]], case["m"], case["n"], case["p"]

    def matrix(rows, cols, col_major, scale_dim):
        shape = (cols, rows) if col_major else (rows, cols)
        if case["dtype"] == "f64":
            x = torch.rand(shape, generator=g, device="cuda", dtype=dt) * 2.0 - 1.0
        else:
            x = torch.randn(shape, generator=g, device="cuda", dtype=dt)
        x = x.t() if col_major else x
        if case["path"] == "fp8":       # every row of A and column of B at its own scale, 10^U(-3, 3)
            u = torch.rand(rows if scale_dim == 0 else cols, generator=g, device="cuda") * 6.0 - 3.0
            x *= (10.0 ** u)[:, None] if scale_dim == 0 else (10.0 ** u)[None, :]
        return x

    A = matrix(m, n, case["a_col"], 0)
    B = matrix(n, p, case["b_col"], 1)
    if case["accumulate"]:
        C = torch.randn((m, p), generator=g, device="cuda", dtype=dt)
    else:
        C = torch.empty((m, p), device="cuda", dtype=dt)
    return A, B, C


def _group_operands(case, seed):
    """Per member (A, B, C, fp8), carved from one buffer of operands and one of results."""
    shapes = _shapes(case)
    pad = lambda x: (x + 63) // 64 * 64  # noqa: E731  (256-byte pieces)
    ops = torch.randn(sum(pad(m * n) + pad(n * p) for m, n, p, _ in shapes), generator=_generator(seed),
                      device="cuda")
    res = torch.zeros(sum(pad(m * p) for m, _, p, _ in shapes), device="cuda")
    out, a, c = [], 0, 0
    for m, n, p, fp8 in shapes:
        A = ops[a:a + m * n].view(m, n)
        a += pad(m * n)
        B = ops[a:a + n * p].view(n, p)
        a += pad(n * p)
        out.append((A, B, res[c:c + m * p].view(m, p), fp8))
        c += pad(m * p)
    return out, res


def prepare(case, seed):
    kind = case["kind"]
    if kind == "gemm":
        A, B, C = _draw_operands(case, seed)
        desc = moa.make_desc(A, B, C, path=case["path"], accumulate=case["accumulate"],
                             flags=moa.MOA_FLAG_FP8_ONE_TERM if case["one_term"] else 0)
        return {"kind": kind, "desc": desc, "C": C, "keep": (A, B)}
    if kind == "group":
        members, res = _group_operands(case, seed)
        descs = [moa.make_desc(A, B, C, path="fp8" if fp8 else "auto") for A, B, C, fp8 in members]
        return {"kind": kind, "descs": descs, "C": res, "keep": members}
    g = _generator(seed)
    if kind == "batched":
        b, m, n, p = case["batch"], case["m"], case["n"], case["p"]
        return {"kind": kind, "A": torch.randn((b, m, n), generator=g, device="cuda"),
                "B": torch.randn((b, n, p), generator=g, device="cuda"), "C": torch.empty((b, m, p), device="cuda")}
    dt, m, n = DTYPES[case["dtype"]], case["m"], case["n"]
    A = torch.randn((m, n), generator=g, device="cuda", dtype=dt)
    if kind == "kronecker":
        B = torch.randn((case["p"], case["q"]), generator=g, device="cuda", dtype=dt)
        C = torch.empty((m * case["p"], n * case["q"]), device="cuda", dtype=dt)
    else:
        B = torch.randn((m, n), generator=g, device="cuda", dtype=dt)
        C = torch.empty((m, n), device="cuda", dtype=dt)
    return {"kind": kind, "A": A, "B": B, "C": C}


def run(state):
    kind = state["kind"]
    if kind == "gemm":
        if moa.moa_gemm_desc_call(state["desc"]) != moa.MOA_OK:
            raise RuntimeError(moa.moa_last_error())
    elif kind == "group":
        moa.moa_gemm_grouped(state["descs"])
    elif kind == "batched":
        moa.moa_gemm_batched(state["A"], state["B"], state["C"])
    elif kind == "kronecker":
        moa.moa_kronecker(state["A"], state["B"], state["C"])
    else:
        moa.moa_hadamard(state["A"], state["B"], state["C"])
    return state["C"]


def work(case):
    """Operands read once, results written once (read too where they are added to); 2 m n p per product."""
    kind = case["kind"]
    if kind == "gemm":
        m, n, p, es = case["m"], case["n"], case["p"], SIZES[case["dtype"]]
        return {"bytes": es * (m * n + n * p + (2 if case["accumulate"] else 1) * m * p), "flops": 2 * m * n * p}
    if kind == "group":
        s = _shapes(case)
        return {"bytes": sum(4 * (m * n + n * p + m * p) for m, n, p, _ in s),
                "flops": sum(2 * m * n * p for m, n, p, _ in s)}
    if kind == "batched":
        b, m, n, p = case["batch"], case["m"], case["n"], case["p"]
        return {"bytes": 4 * b * (m * n + n * p + m * p), "flops": 2 * b * m * n * p}
    es, mn = SIZES[case["dtype"]], case["m"] * case["n"]
    if kind == "kronecker":
        pq = case["p"] * case["q"]
        return {"bytes": es * (mn + pq + mn * pq), "flops": mn * pq}
    return {"bytes": 3 * es * mn, "flops": mn}


def exact(case, seed):
    """The definitions in FP64 (torch), on the inputs of prepare(case, seed)."""
    kind = case["kind"]
    if kind == "gemm":
        A, B, C = _draw_operands(case, seed)
        R = A.double().contiguous() @ B.double().contiguous()
        return R + C.double() if case["accumulate"] else R
    if kind == "group":
        members, res = _group_operands(case, seed)
        out, c = torch.zeros(res.numel(), dtype=torch.float64, device="cuda"), 0
        for A, B, C, _ in members:
            m, p = C.shape
            out[c:c + m * p] = (A.double() @ B.double()).reshape(-1)
            c += (m * p + 63) // 64 * 64
        return out
    s = prepare(case, seed)
    A, B = s["A"].double(), s["B"].double()
    if kind == "batched":
        return torch.stack([A[b] @ B[b] for b in range(A.shape[0])])
    if kind == "kronecker":
        return (A[:, None, :, None] * B[None, :, None, :]).reshape(s["C"].shape)
    return A * B
