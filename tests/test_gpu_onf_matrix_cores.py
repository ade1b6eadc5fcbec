"""The ONF kernel's matrix-core steps against the fma-ordered oracle, bit for
bit: every block, every layout of A and B, sizes at the edges of blocks and of
the LDS stages (whole stages, one k more or less, fewer k than one stage),
overwrite and accumulate, on values where a reordered, padded or flushed step
shows -- subnormals, signed zeros, cancellation -- and with infinities and NaN.
Products whose rows exceed 32-bit offsets run the register-staged kernel.

Every comparison is bitwise (NaN positions equal), so there is no tolerance.
"""
import itertools

import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2306_11148_amd import moa

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
ORACLE = {np.float64: O.gemm_f64_fma, np.float32: O.gemm_f32_fma}


def hard_values(rng, shape, dt):
    """Products and sums of these meet subnormals, -0, cancellation and rounding ties."""
    tiny = -540 if dt == np.float64 else -75          # products near the smallest normal
    x = np.ldexp(rng.integers(-9, 10, shape).astype(np.float64), rng.integers(-3, 4, shape))
    small = rng.random(shape) < 0.3
    x = np.where(small, np.ldexp(rng.standard_normal(shape), tiny + rng.integers(-6, 7, shape)), x)
    return np.where((rng.random(shape) < 0.1), -0.0, x).astype(dt)


def same_bits(got, ref):
    u = np.uint64 if ref.dtype == np.float64 else np.uint32
    nan = np.isnan(ref)
    return np.array_equal(np.isnan(got), nan) and np.array_equal(got.view(u)[~nan], ref.view(u)[~nan])


def place(x, col):
    t = torch.from_numpy(np.ascontiguousarray(x.T if col else x)).to(DEV)
    return t.t() if col else t


@pytest.mark.parametrize("shape", [(1, 1, 1), (31, 32, 33), (33, 31, 65), (64, 129, 63), (129, 7, 130), (96, 97, 257),
                                   (130, 192, 66)])
@pytest.mark.parametrize("dt", [np.float64, np.float32])
def test_every_block_and_layout_bitwise(dt, shape):
    m, n, p = shape
    rng = np.random.default_rng(m * 1000 + n)
    A, B, C0 = (hard_values(rng, s, dt) for s in ((m, n), (n, p), (m, p)))
    A[0, :] = 0.0
    C0[0, :] = -0.0
    ref = {False: ORACLE[dt](A, B), True: ORACLE[dt](A, B, C0, True)}
    for v, a_col, b_col, acc in itertools.product(range(5), (False, True), (False, True), (False, True)):
        At, Bt, Ct = place(A, a_col), place(B, b_col), place(C0, False)
        if v == 4 and (At.stride(0) == 1 and m > 1 and n > 1 and a_col or Bt.stride(0) == 1 and n > 1 and p > 1 and b_col):
            with pytest.raises(moa.MoaError):
                moa.moa_gemm(At, Bt, Ct, path="onf", flags=moa.MOA_FLAG_VARIANT(v))
            continue
        moa.moa_gemm(At, Bt, Ct, path="onf", accumulate=acc, flags=moa.MOA_FLAG_VARIANT(v))
        assert same_bits(Ct.cpu().numpy(), ref[acc]), f"variant {v}, a_col {a_col}, b_col {b_col}, accumulate {acc}"


@pytest.mark.parametrize("dt", [np.float64, np.float32])
def test_infinities_and_nan_stay_in_their_rows_and_columns(dt):
    m, n, p = 70, 37, 67
    rng = np.random.default_rng(8)
    A, B = rng.standard_normal((m, n)).astype(dt), rng.standard_normal((n, p)).astype(dt)
    A[3, 5], A[40, 36], B[7, 9], B[36, 66] = np.inf, np.nan, -np.inf, np.nan
    with np.errstate(all="ignore"):
        ref = ORACLE[dt](A, B)
    for v in range(5):
        Ct = torch.empty((m, p), dtype=torch.from_numpy(A).dtype, device=DEV)
        moa.moa_gemm(place(A, False), place(B, False), Ct, path="onf", flags=moa.MOA_FLAG_VARIANT(v))
        assert same_bits(Ct.cpu().numpy(), ref), f"variant {v}"


@pytest.mark.parametrize("dt,n", [(np.float32, 15_790_327), (np.float64, 7_895_167)])
def test_rows_beyond_32_bit_offsets(dt, n):
    """34 rows of n elements exceed 2^31 bytes: the 64-bit kernel of the same block."""
    g = torch.Generator(device=DEV).manual_seed(3)
    tdt = torch.float64 if dt == np.float64 else torch.float32
    A = torch.randn((3, n), generator=g, device=DEV, dtype=tdt)
    B = torch.randn((n, 2), generator=g, device=DEV, dtype=tdt)
    C = torch.empty((3, 2), device=DEV, dtype=tdt)
    assert 34 * n * A.element_size() >= 2 ** 31 - 1
    moa.moa_gemm(A, B, C, path="onf")
    assert same_bits(C.cpu().numpy(), ORACLE[dt](A.cpu().numpy(), B.cpu().numpy()))
