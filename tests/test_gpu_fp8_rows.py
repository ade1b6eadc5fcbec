"""FP8 conditioning: operands taken by rows and by columns give the same product, bit for bit.

A row-major A (or a column-major B) is conditioned row by row, a wave holding the
row in 4, 8, 16 or 32 registers of four values, longer rows in two passes; a
column-major A (or a row-major B) by columns with its amax in atomics. Exponents
and codes do not depend on the way they were made, so the comparison is bitwise
(no tolerance), at both sides of every register count, at odd lengths and at
addresses that are only 4-byte aligned; a group of two must equal the single calls.
"""
import itertools

import pytest
import torch

from paper_2306_11148_amd import moa

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TERMS = {1: moa.MOA_FLAG_FP8_ONE_TERM, 2: moa.MOA_FLAG_FP8_TWO_TERM}


def operand(x, col, offset):
    """x in the given order, `offset` elements past a 256-byte boundary."""
    rows, cols = x.shape
    buf = torch.empty(rows * cols + offset, device=DEV)[offset:]
    v = buf.view(cols, rows).t() if col else buf.view(rows, cols)
    return v.copy_(x)


def values(g, rows, cols):
    """Normal values; rows and columns of differing magnitude, some of them zero."""
    x = torch.randn(rows, cols, generator=g, device=DEV)
    x *= torch.exp2(torch.randint(-20, 20, (rows, 1), generator=g, device=DEV).float())
    x[rows // 2] = 0.0
    x[:, cols // 3] = 0.0
    return x


@pytest.mark.parametrize("terms", [1, 2])
@pytest.mark.parametrize("n", [1, 2, 63, 65, 255, 257, 1023, 1024, 1025, 2048, 2049, 4096, 4099, 8191, 8192, 8193, 9000])
def test_rows_and_columns_agree(n, terms):
    m, p = 67, 259
    g = torch.Generator(device=DEV).manual_seed(n)
    A, B = values(g, m, n), values(g, p, n).t()
    ref, descs = None, []
    for a_col, b_col in itertools.product((False, True), repeat=2):
        C = torch.full((m, p), float("nan"), device=DEV)
        moa.moa_gemm(operand(A, a_col, n % 4), operand(B, b_col, (n + 1) % 4), C, path="fp8", flags=TERMS[terms])
        ref = C if ref is None else ref
        assert torch.equal(C, ref), f"a_col {a_col}, b_col {b_col}"
    assert torch.isfinite(ref).all()
    a, b = operand(A, False, n % 4), operand(B, False, (n + 3) % 4)
    out = [torch.full((m, p), float("nan"), device=DEV) for _ in range(2)]
    descs = [moa.make_desc(a, b, c, path="fp8", flags=TERMS[terms]) for c in out]
    moa.moa_gemm_grouped(descs)
    for c in out:
        assert torch.equal(c, ref)


@pytest.mark.parametrize("terms", [1, 2])
def test_grouped_members_that_split_k(terms):
    """Members with a split k walk (planned, asked for, more chunks than slabs divide into) beside unsplit ones:
    each bitwise as alone, overwriting and accumulating, p a multiple of four and not, twice in a row."""
    members = [(96, 6000, 132, 0, False), (200, 300, 70, 0, True), (65, 5003, 33, 9, True), (130, 64 * 7, 260, 5, False),
               (3, 4099, 7, 0, True), (64, 65, 64, 2, False), (33, 40, 129, 0, False), (1, 9000, 1, 64, True)]
    g = torch.Generator(device=DEV).manual_seed(terms)
    ops, descs = [], []
    for m, n, p, chunks, acc in members:
        flags = TERMS[terms] | (moa.MOA_FLAG_SPLIT_K(chunks) if chunks else 0)
        A, B, C0 = values(g, m, n), values(g, n, p), torch.randn(m, p, generator=g, device=DEV)
        R, C = C0.clone(), torch.empty_like(C0)
        moa.moa_gemm(A, B, R, path="fp8", accumulate=acc, flags=flags)
        ops.append((C, C0, R, A, B))
        descs.append(moa.make_desc(A, B, C, path="fp8", accumulate=acc, flags=flags))
    for _ in range(2):
        for C, C0, *_ in ops:
            C.copy_(C0)
        moa.moa_gemm_grouped(descs)
        for k, (C, _, R, *_) in enumerate(ops):
            assert torch.equal(C, R), f"member {k}"


def test_walks_longer_than_one_grid_of_bands():
    """n past 65536 bands of 64 rows (a grid's y extent): columns of a row-major B against a column-major one."""
    m, n, p = 3, 65536 * 64 + 77, 5
    g = torch.Generator(device=DEV).manual_seed(0)
    A, B = torch.randn(m, n, generator=g, device=DEV), torch.randn(p, n, generator=g, device=DEV)
    B[:, -1] = 100.0                                            # the amax of every column is in the last band
    out = []
    for b_col in (False, True):
        C = torch.full((m, p), float("nan"), device=DEV)
        moa.moa_gemm(A, operand(B.t(), b_col, 0), C, path="fp8", flags=TERMS[1])
        out.append(C)
    assert torch.isfinite(out[0]).all() and torch.equal(out[0], out[1])


def test_exponents_of_more_rows_than_one_grid():
    """More rows than the row-exponent kernel's workgroups, which then take several."""
    m, n = (1 << 20) + 3, 2
    g = torch.Generator(device=DEV).manual_seed(1)
    A, B = torch.randn(m, n, generator=g, device=DEV), torch.randn(n, 3, generator=g, device=DEV)

    def exponents(X):
        u8 = dict(dtype=torch.uint8, device=DEV)
        e, f = (torch.full((k,), 999, dtype=torch.int32, device=DEV) for k in (X.shape[0], 3))
        moa.moa_quantise_fp8(X, B, e, torch.empty(X.shape, **u8), f, torch.empty(B.shape, **u8))
        return e

    e = exponents(A)
    for at in (0, (1 << 20) - 500, m - 1000):
        assert torch.equal(e[at:at + 1000], exponents(A[at:at + 1000].contiguous()))
