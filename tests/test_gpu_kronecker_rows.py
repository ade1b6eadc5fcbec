"""Kronecker products at the edges of the kernel's row runs and column chunks, bitwise against the oracle.

Row runs that start inside a row of A, p = 1 and m = 1 (i or k changes every row
or never), columns of exactly one chunk and one more, vector widths that q or C's
or B's alignment rule out, in both types, overwrite and accumulate. Each element
is one rounded product (and one rounded sum), so there is no tolerance.
"""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2306_11148_amd import moa

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def device(x, offset):
    buf = torch.empty(x.size + offset, dtype=torch.from_numpy(x).dtype, device=DEV)[offset:]
    return buf.view(x.shape).copy_(torch.from_numpy(x))


@pytest.mark.parametrize("shape", [(1, 1, 1, 1), (1, 7, 9, 4), (9, 3, 1, 8), (5, 16, 7, 64), (3, 257, 5, 4),
                                   (2, 41, 3, 25), (700, 3, 6, 12)])
@pytest.mark.parametrize("dt", [np.float32, np.float64])
@pytest.mark.parametrize("offset", [0, 1])
def test_bitwise(shape, dt, offset):
    m, n, p, q = shape
    rng = np.random.default_rng(m + n + p + q)
    A, B = rng.standard_normal((m, n)).astype(dt), rng.standard_normal((p, q)).astype(dt)
    C0 = rng.standard_normal((m * p, n * q)).astype(dt)
    for acc in (False, True):
        Ct = device(C0 if acc else np.full_like(C0, np.nan), offset)
        moa.moa_kronecker(device(A, offset), device(B, offset), Ct, accumulate=acc)
        ref = O.kronecker(A, B, C0, True) if acc else O.kronecker(A, B)
        assert np.array_equal(Ct.cpu().numpy(), ref), f"accumulate {acc}"


# rows of C in whole vectors where q or B's alignment rules the wide form out, and runs of one, two, four and more rows
@pytest.mark.parametrize("shape", [(2, 4, 3, 5), (3, 64, 5, 31), (1, 4, 9000, 3), (1100, 2, 2, 6), (33, 8, 129, 9),
                                   (5, 4, 7, 8), (2, 682, 3, 3), (2, 341, 700, 6)])
@pytest.mark.parametrize("dt", [np.float32, np.float64])
@pytest.mark.parametrize("b_offset", [0, 1])
def test_gathered_rows_and_runs(shape, dt, b_offset):
    m, n, p, q = shape
    rng = np.random.default_rng(m + n + p + q)
    A, B = rng.standard_normal((m, n)).astype(dt), rng.standard_normal((p, q)).astype(dt)
    C0 = rng.standard_normal((m * p, n * q)).astype(dt)
    for acc in (False, True):
        Ct = device(C0 if acc else np.full_like(C0, np.nan), 0)
        moa.moa_kronecker(device(A, 1), device(B, b_offset), Ct, accumulate=acc)
        ref = O.kronecker(A, B, C0, True) if acc else O.kronecker(A, B)
        assert np.array_equal(Ct.cpu().numpy(), ref), f"accumulate {acc}"
