"""Record packers at every alignment: row-major and column-major operands give the same bits.

A row-major A goes through the row packer and a column-major one, whose values
are the same, through the transposing packer (B the other way round); records do
not depend on the way they were made, so products are compared bitwise, at odd
lengths and at addresses that are only 4-byte aligned.
"""
import itertools

import pytest
import torch

from paper_2306_11148_amd import moa

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("path", ["split_bf16", "mfma_f32"])
@pytest.mark.parametrize("shape", [(1, 1, 1), (17, 15, 65), (65, 33, 63), (130, 67, 131), (64, 72, 64), (300, 259, 261)])
def test_rows_and_columns_agree(path, shape):
    m, n, p = shape
    g = torch.Generator(device=DEV).manual_seed(m * n)
    A, B = torch.randn(m, n, generator=g, device=DEV), torch.randn(n, p, generator=g, device=DEV)
    ref = None
    for a_col, b_col, offset in itertools.product((False, True), (False, True), (0, 1, 2, 3)):
        def at(x, col):
            v = torch.empty(x.numel() + offset, device=DEV)[offset:]
            return (v.view(x.shape[1], x.shape[0]).t() if col else v.view(x.shape)).copy_(x)
        C = torch.full((m, p), float("nan"), device=DEV)
        moa.moa_gemm(at(A, a_col), at(B, b_col), C, path=path, flags=moa.MOA_FLAG_VARIANT(0))
        ref = C if ref is None else ref
        assert torch.equal(C, ref), f"a_col {a_col}, b_col {b_col}, offset {offset}"
    bound = 2e-5 * (A.double().abs() @ B.double().abs())       # both paths hold 1e-5 normwise
    assert ((ref.double() - A.double() @ B.double()).abs() <= bound).all()


@pytest.mark.parametrize("path", ["split_bf16", "fp8"])
@pytest.mark.parametrize("accumulate", [False, True])
def test_rows_of_c_beyond_buffer_offsets(path, accumulate):
    """p at and past 2^26, where C is written with 64-bit addresses: the same bits as a narrow slice of the product."""
    for p in ((1 << 26) - 1, (1 << 26) + 5):
        m, n, w = 9, 3, 300
        g = torch.Generator(device=DEV).manual_seed(p)
        A, B = torch.randn(m, n, generator=g, device=DEV), torch.randn(n, p, generator=g, device=DEV)
        C = torch.ones(m, p, device=DEV)
        moa.moa_gemm(A, B, C, path=path, accumulate=accumulate, flags=moa.MOA_FLAG_VARIANT(0))
        for at in (0, p // 2, p - w):
            R = torch.ones(m, w, device=DEV)
            moa.moa_gemm(A, B[:, at:at + w].contiguous(), R, path=path, accumulate=accumulate,
                         flags=moa.MOA_FLAG_VARIANT(0))
            assert torch.equal(C[:, at:at + w], R), f"p {p}, columns from {at}"
