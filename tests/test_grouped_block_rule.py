"""Grouped split-BF16: the static rule's block on groups whose times under every block were measured.

Large groups pay for every slab step (128 x 128 blocks, variant 2); a few products with long walks leave compute
units idle and take small blocks (variant 1).
"""
import math
import random

import pytest

from paper_2306_11148_amd import moa


def mixed(count, seed):
    """Log-uniform m, p in 64 .. 2048 and n in 64 .. 4096."""
    r = random.Random(seed)
    log = lambda lo, hi: int(round(math.exp(r.uniform(math.log(lo), math.log(hi)))))  # noqa: E731
    out = []
    for _ in range(count):
        out.append((log(64, 2048), log(64, 4096), log(64, 2048)))
        r.randrange(100)
    return out


@pytest.mark.parametrize("shapes,variant", [
    (mixed(64, 45), 2),                     # us with variants 1 .. 4: 348, 232, 271, 353
    (mixed(64, 69), 2),                     # 329, 256, 268, 353
    (mixed(31, 60), 2),                     # 210, 186, 194, 255
    ([(861, 681, 259)] * 17, 2),            # 84, 57, 67, 67
    ([(293, 1001, 675)] * 50, 2),           # 199, 136, 150, 174
    (mixed(4, 66), 1),                      # 79, 110, 90, 103
    ([(137, 67, 1192)] * 43, 2),            # 75, 48, 59, 73: short k walks
    ([(159, 50, 613)] * 111, 2),            # 79, 49, 61, 75
    ([(43, 14, 967)] * 62, 3),              # 64, 40.3, 39.5, 64
])
def test_measured_best_block(shapes, variant):
    descs = []
    for k, (m, n, p) in enumerate(shapes):
        A = 0x100000000 + k * 3 * (1 << 26)
        descs.append(moa.moa_gemm_desc(m=m, n=n, p=p, dtype=moa.MOA_F32, path=moa.MOA_PATH_AUTO, A=A, B=A + (1 << 26),
                                       C=A + 2 * (1 << 26)))
    assert moa.moa_grouped_plan_query(descs)["variant"] == variant
