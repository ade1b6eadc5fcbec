"""Scaled FP8 of a tall product with a column-major B: the rows of A and the columns of B are conditioned in one
launch, which together pass the 2^32 threads that a grid holds in x. Sampled blocks of rows, bitwise the product of
those rows alone (every row has its own exponent, every element its own sum).
"""
import pytest
import torch

from paper_2306_11148_amd import moa


@pytest.mark.gpu
def test_rows_of_both_operands_beyond_one_grid_extent():
    m, n, p = 2 ** 26 - 16, 3, 32                   # 2^24 - 4 workgroups of four rows of A, 8 of B
    g = torch.Generator(device="cuda:0").manual_seed(6)
    A = torch.randn((m, n), generator=g, device="cuda:0")
    B = torch.randn((p, n), generator=g, device="cuda:0").t()
    C = torch.full((m, p), float("nan"), device="cuda:0")
    moa.moa_gemm(A, B, C, path="fp8", flags=moa.MOA_FLAG_FP8_ONE_TERM)
    for r in (0, m // 2 - 7, 2 ** 24 * 3 + 5, m - 128):
        R = torch.empty((128, p), device="cuda:0")
        moa.moa_gemm(A[r:r + 128], B, R, path="fp8", flags=moa.MOA_FLAG_FP8_ONE_TERM)
        assert torch.equal(C[r:r + 128], R), f"rows from {r}"
    assert not torch.isnan(C).any()
