"""Autotuner records and split-BF16 products that run without conditioning: a record moves a product off that kernel
only where a record-ring block was timed faster than it."""
import pytest
import torch

from paper_2306_11148_amd import moa


def direct(m, n, p):
    return moa.moa_plan_query(moa.moa_gemm_desc(m=m, n=n, p=p, dtype=moa.MOA_F32, path=moa.MOA_PATH_SPLIT_BF16, A=None,
                                                B=None, C=None, accumulate=0, flags=0))


@pytest.mark.parametrize("shape,record", [((192, 320, 160), "1 3 1 8 9 8 0"), ((512, 32768, 512), "1 3 1 9 15 9 0")])
@pytest.mark.parametrize("tail,kept", [(" 0.05\n", True), (" 0.05 1\n", True), (" 0.05 0\n", False)])
def test_records_of_a_file(tmp_path, shape, record, tail, kept):
    assert direct(*shape)["path"] == int(record.split()[1])
    moa.moa_autotune_clear()
    try:
        f = tmp_path / "tune.txt"
        f.write_text("# moa autotune v1\n" + record + tail)
        moa.moa_autotune_load(str(f))
        q = direct(*shape)
        assert q["tuned"] == 1 and q["variant"] == 0 and (q["direct_block"] != 0) == kept
        moa.moa_autotune_save(str(f))
        moa.moa_autotune_clear()
        moa.moa_autotune_load(str(f))
        assert direct(*shape) == q
    finally:
        moa.moa_autotune_clear()


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(192, 320, 160), (512, 32768, 512)])
def test_tuning_keeps_the_faster_kernel(shape):
    """Both run in a third to two thirds of the time of the best record-ring block."""
    m, n, p = shape
    A, B, C = (torch.randn(s, device="cuda:0") for s in ((m, n), (n, p), (m, p)))
    moa.moa_autotune_clear()
    try:
        before = direct(m, n, p)
        ring = min(_time(A, B, C, v) for v in range(4))
        plan, ms = moa.moa_autotune(moa.make_desc(A, B, C, path="split_bf16"), reps=20)
        assert plan["tuned"] == 1 and plan["direct_block"] == before["direct_block"] != 0
        assert ms < ring
    finally:
        moa.moa_autotune_clear()


def _time(A, B, C, variant, reps=20):
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    for k in range(reps + 1):
        if k == 1:
            e0.record()
        moa.moa_gemm(A, B, C, path="split_bf16", flags=moa.MOA_FLAG_VARIANT(variant))
    e1.record()
    e1.synchronize()
    return e0.elapsed_time(e1) / reps
