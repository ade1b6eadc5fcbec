"""Two-term FP8 default block: 128 x 128 or a rectangle, whichever takes fewer rounds of the 256 CUs."""
import pytest

from paper_2306_11148_amd import moa


@pytest.mark.parametrize("m,p,tile", [
    (1024, 1024, (128, 128)),       # 64 blocks
    (2048, 2048, (128, 128)),       # one round of either: 1 against 1.75
    (2560, 2560, (128, 256)),       # 2 rounds against 1.75
    (3072, 3072, (128, 128)),       # 3 rounds against 3.5
    (3001, 1999, (128, 256)),       # 2 rounds against 1.75
    (8192, 8192, (128, 256)),       # 16 rounds against 14
    (65536, 128, (256, 128)),       # the tall rectangle fits: 2 rounds against 1.75
    (128, 65536, (128, 256)),
])
def test_two_term_default_block(m, p, tile):
    d = moa.moa_gemm_desc(A=1, B=1, C=1, m=m, n=1024, p=p, dtype=moa.MOA_F32, path=moa.MOA_PATH_FP8_SCALED)
    q = moa.moa_plan_query(d)
    assert (q["tile_m"], q["tile_n"]) == tile
