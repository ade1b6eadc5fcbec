"""Split-BF16 products without a conditioning pass against the conditioned record ring, bit for bit.

The default plan of a product of few blocks splits the FP32 operands on the way
through LDS; MOA_FLAG_VARIANT(0) keeps the record ring. Both give every element
the same operation sequence, so the comparison is bitwise (no tolerance): every
layout of A, B and C, overwrite and accumulate, shapes at the edges of the 64
and 128 blocks, k walks of one slab, an odd and an even number of slabs, part of
a slab, operands at every alignment their type allows, and shapes that take each
of the four blocks (chosen by the busiest compute unit's load).
"""
import itertools

import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2306_11148_amd import moa

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def operand(g, rows, cols, col, offset=0):
    """rows x cols, row- or column-major, `offset` elements past a 256-byte boundary."""
    buf = torch.randn(rows * cols + offset, generator=g, device=DEV)[offset:]
    return buf.view(cols, rows).t() if col else buf.view(rows, cols)


def both(A, B, C0, accumulate):
    out = []
    for flags in (0, moa.MOA_FLAG_VARIANT(0)):
        C = torch.empty_strided(C0.shape, C0.stride(), device=DEV)
        C.copy_(C0 if accumulate else torch.full_like(C0, float("nan")))
        moa.moa_gemm(A, B, C, path="split_bf16", accumulate=accumulate, flags=flags)
        out.append(C)
    return out


@pytest.mark.parametrize("shape", [(1, 1, 1), (63, 16, 65), (64, 17, 64), (65, 15, 63), (127, 32, 129), (129, 47, 128),
                                   (130, 33, 257), (200, 700, 90), (2, 4095, 3)])
def test_layouts_and_edges(shape):
    m, n, p = shape
    g = torch.Generator(device=DEV).manual_seed(m + n + p)
    for a_col, b_col, c_col, acc in itertools.product((False, True), repeat=4):
        A, B, C0 = operand(g, m, n, a_col), operand(g, n, p, b_col), operand(g, m, p, c_col)
        got, ref = both(A, B, C0, acc)
        assert torch.equal(got, ref), f"a_col {a_col}, b_col {b_col}, c_col {c_col}, accumulate {acc}"


@pytest.mark.parametrize("offset", [1, 2, 3])
def test_unaligned_operands(offset):
    g = torch.Generator(device=DEV).manual_seed(offset)
    for a_col, b_col in itertools.product((False, True), repeat=2):
        A, B = operand(g, 131, 75, a_col, offset), operand(g, 75, 133, b_col, offset)
        C0 = operand(g, 131, 133, False, offset)
        got, ref = both(A, B, C0, True)
        assert torch.equal(got, ref)


# 64 x 64 (49 blocks), 64 x 128 and 128 x 64 (480 blocks of 64 x 64 would be two
# per compute unit), 128 x 128 (256 blocks), and past the rule (record ring both times)
@pytest.mark.parametrize("shape", [(448, 100, 448), (1530, 65, 1236), (1920, 40, 1024), (2000, 48, 2040),
                                   (3584, 33, 3600)])
def test_every_block_of_the_rule(shape):
    m, n, p = shape
    g = torch.Generator(device=DEV).manual_seed(9)
    A, B, C0 = operand(g, m, n, False), operand(g, n, p, False), operand(g, m, p, False)
    got, ref = both(A, B, C0, False)
    assert torch.equal(got, ref)
    rows = [0, m // 2, m - 1]
    R = O.gemm_f64(A[rows].cpu().numpy().astype(np.float64), B.cpu().numpy().astype(np.float64))
    assert O.rel_err(got[rows].cpu().numpy(), R) <= 1e-5


@pytest.mark.parametrize("shape,chunks", [((1, 33, 1), 3), ((130, 1000, 67), 2), ((129, 4096, 257), 0), ((64, 20000, 64), 0),
                                          ((300, 5003, 132), 7)])
def test_split_k_layouts(shape, chunks):
    """Chunks of the k walk, asked for or planned: the same partials and sums as the record ring's."""
    m, n, p = shape
    g = torch.Generator(device=DEV).manual_seed(n)
    for a_col, b_col, c_col, acc in itertools.product((False, True), repeat=4):
        A, B, C0 = operand(g, m, n, a_col), operand(g, n, p, b_col), operand(g, m, p, c_col)
        out = []
        for flags in (0, moa.MOA_FLAG_VARIANT(0)):
            C = torch.empty_strided(C0.shape, C0.stride(), device=DEV)
            C.copy_(C0 if acc else torch.full_like(C0, float("nan")))
            moa.moa_gemm(A, B, C, path="split_bf16", accumulate=acc, flags=flags | moa.MOA_FLAG_SPLIT_K(chunks))
            out.append(C)
        assert torch.equal(out[0], out[1]), f"a_col {a_col}, b_col {b_col}, c_col {c_col}, accumulate {acc}"


def test_grouped_split_k_members_share_the_launch():
    """Members that split k (planned, asked for, ragged, accumulating), unsplit ones and an FP8 one that splits:
    each bitwise as alone, whichever persistent kernel runs, twice in a row on the same scratch."""
    members = [(96, 6000, 130, "split_bf16", 0, False), (300, 700, 200, "split_bf16", 0, False),
               (65, 5003, 33, "split_bf16", moa.MOA_FLAG_SPLIT_K(9), True), (3, 4099, 7, "split_bf16", 0, True),
               (128, 40, 64, "split_bf16", moa.MOA_FLAG_SPLIT_K(2), False), (96, 4500, 70, "fp8", 0, False)]
    g = torch.Generator(device=DEV).manual_seed(2)
    ops, descs = [], []
    for m, n, p, path, flags, acc in members:
        A, B, C0 = operand(g, m, n, False), operand(g, n, p, False), operand(g, m, p, False)
        R = C0.clone()
        moa.moa_gemm(A, B, R, path=path, accumulate=acc, flags=flags)
        C = torch.empty_like(C0)
        ops.append((A, B, C, C0, R))
        descs.append(moa.make_desc(A, B, C, path=path, accumulate=acc, flags=flags))
    assert moa.moa_grouped_plan_query(descs)["persistent_members"] == 5
    for variant in (-1, *range(moa.MOA_GROUPED_VARIANTS), -1):
        for _, _, C, C0, _ in ops:
            C.copy_(C0)
        moa.moa_gemm_grouped_variant(descs, variant)
        for k, (_, _, C, _, R) in enumerate(ops):
            assert torch.equal(C, R), f"variant {variant}, member {k}"
