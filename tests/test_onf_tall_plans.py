"""Tall and wide ONF products: which row counts the default plan takes, and rows far down a tall product.

The default block may be any of the table, but how many rows a product may have
does not depend on it: 65535 blocks of the largest block of its type and layout
(128 rows; 64 for FP64 with a column-major operand). A launch holds fewer than
2^32 threads in x, so the block has to leave fewer than 2^24 workgroups.
"""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2306_11148_amd import inputs, moa

F64, F32 = moa.MOA_F64, moa.MOA_F32


def plan(m, n, p, dtype, flags=0):
    return moa.moa_plan_query(moa.moa_gemm_desc(m=m, n=n, p=p, dtype=dtype, path=moa.MOA_PATH_ONF, A=None, B=None, C=None,
                                                accumulate=0, flags=flags))


@pytest.mark.parametrize("dtype", [F64, F32])
@pytest.mark.parametrize("n", [1, 16, 4096])
@pytest.mark.parametrize("p", [1, 16, 32, 33, 64, 96, 128, 200, 300, 512])
def test_rows_up_to_the_largest_blocks_limit(dtype, n, p):
    for m in (65535 * 32, 65535 * 32 + 1, 3000000, 65535 * 64 + 1, 8000000, 65535 * 128):
        assert plan(m, n, p, dtype)["path"] == moa.MOA_PATH_ONF
    with pytest.raises(moa.MoaError) as e:
        plan(65535 * 128 + 1, n, p, dtype)
    assert e.value.status == moa.MOA_ERR_SHAPE


@pytest.mark.parametrize("flag", [moa.MOA_FLAG_A_COL, moa.MOA_FLAG_B_COL])
@pytest.mark.parametrize("dtype,rows", [(F64, 64), (F32, 128)])
def test_column_major_operands(dtype, rows, flag):
    plan(65535 * rows, 16, 16, dtype, flag)
    with pytest.raises(moa.MoaError) as e:
        plan(65535 * rows + 1, 16, 16, dtype, flag)
    assert e.value.status == moa.MOA_ERR_SHAPE


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_rows_of_a_tall_product(dtype):
    """2097223 rows: beyond 65535 blocks of 32. Rows at the start, around that limit and at the end, bitwise."""
    m, n, p = 65535 * 32 + 103, 21, 16
    g = torch.Generator(device="cuda:0").manual_seed(3)
    A = torch.randn((m, n), generator=g, device="cuda:0", dtype=torch.float64 if dtype == np.float64 else torch.float32)
    _, B = inputs.uniform_f64(1, n, p, seed=4)
    B = B.astype(dtype)
    C = torch.full((m, p), float("nan"), device="cuda:0", dtype=A.dtype)
    moa.moa_gemm(A, torch.from_numpy(B).to("cuda:0"), C, path="onf")
    assert not torch.isnan(C).any()
    rows = torch.tensor([0, 1, m // 2, 65535 * 32 - 1, 65535 * 32, 65535 * 32 + 1, m - 2, m - 1], device="cuda:0")
    fma = O.gemm_f64_fma if dtype == np.float64 else O.gemm_f32_fma
    assert np.array_equal(C[rows].cpu().numpy(), fma(np.ascontiguousarray(A[rows].cpu().numpy()), B))


@pytest.mark.parametrize("dtype", [F64, F32])
@pytest.mark.parametrize("m", [1, 32, 33])
@pytest.mark.parametrize("p", [2 ** 24, 2 ** 29 - 1, 2 ** 29, 2 ** 29 + 5, 2 ** 30, 2 ** 30 + 5])
def test_wide_products_fit_the_grid(dtype, m, p):
    q = plan(m, 1, p, dtype)
    assert q["workgroups"] * q["threads"] < 2 ** 32


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,p", [(torch.float64, 2 ** 29 + 5), (torch.float32, 2 ** 30 + 5)])
def test_a_wide_product(dtype, p):
    """One row, k of one step: C[0][j] = A[0][0] B[0][j], one rounding."""
    A = torch.tensor([[1.1]], device="cuda:0", dtype=dtype)
    B = torch.randn((1, p), generator=torch.Generator(device="cuda:0").manual_seed(5), device="cuda:0", dtype=dtype)
    C = torch.full((1, p), float("nan"), device="cuda:0", dtype=dtype)
    moa.moa_gemm(A, B, C, path="onf")
    assert torch.equal(C, B * A)
