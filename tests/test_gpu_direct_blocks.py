"""Every block of the split-BF16 kernel without conditioning, in every layout of A and B, overwrite and accumulate,
operands on 16-byte boundaries and off them: bitwise the record ring (the same sequence of operations per element).
The plan says which block runs, so a change of the rule cannot leave one out unseen."""
import itertools

import pytest
import torch

from paper_2306_11148_amd import moa

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def operand(g, rows, cols, col, offset):
    buf = torch.randn(rows * cols + offset, generator=g, device=DEV)[offset:]
    return buf.view(cols, rows).t() if col else buf.view(rows, cols)


@pytest.mark.parametrize("offset", [0, 1, 3])
@pytest.mark.parametrize("shape,block", [((130, 33, 257), (64, 64)), ((1530, 65, 1236), (64, 128)),
                                         ((384, 65, 5440), (128, 64)), ((2000, 47, 2039), (128, 128))])
def test_layouts_of_every_block(shape, block, offset):
    m, n, p = shape
    g = torch.Generator(device=DEV).manual_seed(offset)
    for a_col, b_col, acc in itertools.product((False, True), repeat=3):
        A, B, C0 = operand(g, m, n, a_col, offset), operand(g, n, p, b_col, offset), operand(g, m, p, False, offset)
        out = []
        for flags in (0, moa.MOA_FLAG_VARIANT(0)):
            C = torch.full((m * p + offset,), float("nan"), device=DEV)[offset:].view(m, p)
            if acc:
                C.copy_(C0)
            desc = moa.make_desc(A, B, C, path="split_bf16", accumulate=acc, flags=flags)
            ran = moa.moa_plan_query(desc)["direct_block"]
            assert (ran >> 16, ran & 0xFFFF) == ((0, 0) if flags else block)
            moa.moa_gemm(A, B, C, path="split_bf16", accumulate=acc, flags=flags)
            out.append(C)
        assert torch.equal(out[0], out[1]), f"a_col {a_col}, b_col {b_col}, accumulate {acc}"
