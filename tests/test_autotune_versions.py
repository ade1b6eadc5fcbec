"""Grouped autotuner records of older files name kernels that have been replaced: they are passed over."""
import pytest

from paper_2306_11148_amd import moa


def query():
    descs = []
    for k in range(8):
        A = 0x100000000 + k * 3 * (1 << 26)
        descs.append(moa.moa_gemm_desc(m=64, n=300, p=256, dtype=moa.MOA_F32, path=moa.MOA_PATH_AUTO, A=A, B=A + (1 << 26),
                                       C=A + 2 * (1 << 26)))
    return moa.moa_grouped_plan_query(descs)


def test_grouped_records_of_the_first_format(tmp_path):
    record, single = "1 16 3 6 9 8 1 0.25\n", "0 1 1 8 8 8 2 0.5\n"
    f64 = moa.moa_gemm_desc(m=256, n=256, p=256, dtype=moa.MOA_F64, path=moa.MOA_PATH_ONF)
    f = tmp_path / "group.txt"
    moa.moa_autotune_clear()
    try:
        f.write_text("# moa autotune v1: dtype path terms log2m log2n log2p variant ms\n" + record + single)
        moa.moa_autotune_load(str(f))
        assert query()["tuned"] == 0
        assert moa.moa_plan_query(f64)["tuned"] == 1            # single products' blocks are the same
        f.write_text("# moa autotune v1\n1 16 3 6 9 8 5 0.25\n")  # still checked
        with pytest.raises(moa.MoaError):
            moa.moa_autotune_load(str(f))
        f.write_text(record)
        moa.moa_autotune_load(str(f))
        assert query()["tuned"] == 1 and query()["variant"] == 1
        moa.moa_autotune_save(str(f))
        moa.moa_autotune_clear()
        moa.moa_autotune_load(str(f))                           # a file written now keeps them
        assert query()["tuned"] == 1 and query()["variant"] == 1
    finally:
        moa.moa_autotune_clear()
