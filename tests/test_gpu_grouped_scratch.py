"""Grouped members that split their k walk: a large group needs no more scratch at once than a gigabyte or its largest
member, and every result stays bitwise the single product's."""
import pytest
import torch

from paper_2306_11148_amd import moa

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("path,flags", [("split_bf16", 0), ("fp8", moa.MOA_FLAG_FP8_ONE_TERM)])
def test_scratch_of_a_group_with_large_partials(path, flags):
    """24 members of 171 (FP8: 128) chunks of 4 MiB: 16 and 12 GiB of partials together; and small ones among them."""
    g = torch.Generator(device=DEV).manual_seed(8)
    shapes = [(1024, 8192, 1024, flags | moa.MOA_FLAG_SPLIT_K(255))] * 24
    for at in (0, 5, 26):
        shapes.insert(at, (130, 100, 70, flags))
        shapes.insert(at, (96, 6000, 130, flags))
    A = torch.randn((1024, 8192), generator=g, device=DEV)
    B = torch.randn((8192, 1024), generator=g, device=DEV)
    descs, out = [], []
    for k, (m, n, p, fl) in enumerate(shapes):
        X, Y = (A, B) if n == 8192 else (A.view(-1)[64 * k:64 * k + m * n].view(m, n), B.view(-1)[:n * p].view(n, p))
        C = torch.full((m, p), float("nan"), device=DEV)
        out.append((X, Y, C, fl))
        descs.append(moa.make_desc(X, Y, C, path=path, flags=fl))
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    moa.moa_gemm_grouped(descs)
    torch.cuda.synchronize()
    assert before - torch.cuda.mem_get_info()[0] < 4 << 30
    for k, (X, Y, C, fl) in enumerate(out):
        R = torch.empty_like(C)
        moa.moa_gemm(X, Y, R, path=path, flags=fl)
        assert torch.equal(C, R), f"member {k}"
