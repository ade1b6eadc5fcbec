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
