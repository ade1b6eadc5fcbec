"""ONF default blocks where the time of every block was measured: short k walks over a large C take large blocks, long
ones the block that spreads best."""
import pytest

from paper_2306_11148_amd import moa

F64, F32 = moa.MOA_F64, moa.MOA_F32


@pytest.mark.parametrize("dtype,shape,acc,variants", [
    (F64, (6000, 30, 6000), 0, (4,)),           # us with variants 0, 1, 2, 4: 111, 123, 81, 75
    (F64, (6000, 100, 6000), 1, (4,)),          # 254, 247, 213, 186
    (F64, (100000, 16, 128), 0, (2, 4)),        # 37, 39, 29, 29
    (F64, (300000, 8, 64), 0, (4,)),            # 51, 51, 49, 40
    (F64, (500000, 16, 16), 0, (0,)),           # 45, 93, 88, 71
    (F32, (100000, 16, 128), 1, (2,)),          # 25, 22, 19, 21
    (F32, (300000, 64, 64), 0, (1,)),           # 41, 36, 57, 57
    (F32, (6000, 30, 6000), 0, (2,)),           # 56, 47, 37, 42
    (F64, (1999, 1531, 2113), 1, (0,)), (F64, (256, 256, 256), 0, (0,)), (F32, (8192, 8192, 8192), 0, (4,)),
])
def test_default_block(dtype, shape, acc, variants):
    m, n, p = shape
    q = moa.moa_plan_query(moa.moa_gemm_desc(m=m, n=n, p=p, dtype=dtype, path=moa.MOA_PATH_ONF, A=None, B=None, C=None,
                                             accumulate=acc, flags=0))
    assert q["variant"] in variants
