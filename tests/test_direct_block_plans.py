"""moa_plan_query names the block of split-BF16 products that run without conditioning."""
import pytest

from paper_2306_11148_amd import moa


def plan(m, n, p, flags=0, path=moa.MOA_PATH_SPLIT_BF16):
    return moa.moa_plan_query(moa.moa_gemm_desc(m=m, n=n, p=p, dtype=moa.MOA_F32, path=path, A=None, B=None, C=None,
                                                accumulate=0, flags=flags))


@pytest.mark.parametrize("shape,block", [
    ((192, 320, 160), (64, 64)), ((1530, 65, 1236), (64, 128)), ((384, 65, 5440), (128, 64)),
    ((2000, 48, 2040), (128, 128)), ((512, 32768, 512), (128, 128)), ((8192, 8192, 8192), (0, 0)),
    ((3072, 3072, 3072), (0, 0))])
def test_block_that_runs(shape, block):
    q = plan(*shape)
    assert (q["direct_block"] >> 16, q["direct_block"] & 0xFFFF) == block
    assert plan(*shape, flags=moa.MOA_FLAG_VARIANT(0))["direct_block"] == 0      # the record ring, asked for
    assert plan(*shape, path=moa.MOA_PATH_FP8_SCALED)["direct_block"] == 0


def test_column_major_result_is_planned_transposed():
    q = plan(5440, 65, 384, flags=moa.MOA_FLAG_C_COL)
    assert (q["direct_block"] >> 16, q["direct_block"] & 0xFFFF) == (128, 64)


@pytest.mark.parametrize("flags", range(8))
@pytest.mark.parametrize("shape", [(1, 1, 1), (63, 16, 65), (65, 17, 63), (130, 33, 257), (192, 320, 160), (384, 65, 5440),
                                   (1530, 65, 1236), (2000, 48, 2040), (100, 20000, 100), (3, 16 * 131071, 5),
                                   (1000, 4, 90000)])
def test_direct_loads_stay_in_bounds(shape, flags):
    """Every load of the kernel that runs, in every layout: inside the operand and its 32-bit offsets, and covering
    what the block needs."""
    d = moa.moa_gemm_desc(m=shape[0], n=shape[1], p=shape[2], dtype=moa.MOA_F32, path=moa.MOA_PATH_SPLIT_BF16, A=None,
                          B=None, C=None, accumulate=0, flags=flags << 24)
    q = moa.moa_plan_query(d)
    loads, bad = moa.moa_diag_ring_loads(d)
    assert loads > 0 and bad == 0
    if q["direct_block"] and q["split_k"] == 1:
        m, p = (shape[2], shape[0]) if flags & 4 else (shape[0], shape[2])
        rows, cols = q["direct_block"] >> 16, q["direct_block"] & 0xFFFF
        assert loads == -(-m // rows) * rows // 16 + -(-p // cols) * cols // 16
