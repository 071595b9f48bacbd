"""bf16 decode of few rows: fewer tiles than waves (one tile a wave for short
segments, up to four for long ones, the waves spread over the workgroups), and
segments cut into so many pieces that the merge's waves share them. Against the
oracle at the bf16 bar of every other kernel test, and twice bitwise."""

import numpy as np
import pytest

from paper_2504_09590_amd import workload as W
from tests.gpu_helpers import announce, compare, poison_unowned, require_gpu
from tests.test_gpu_decode import ref_decode, run_decode

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("group,hkv", [(1, 8), (2, 2), (4, 8), (8, 1)])
# blocks per segment around the limits: 1, 16 (one tile a wave below 32 blocks), 17 and 33 pieces a segment, and
# 64, 68 (four tiles a wave, 16 and 17 pieces), 1000
@pytest.mark.parametrize("blocks", [1, 16, 17, 33, 64, 68, 1000])
def test_one_row(group, hkv, blocks):
    require_gpu()
    ctx = 16 * blocks - (blocks % 3)
    b = poison_unowned(W.custom([ctx], [W.BE], group * hkv, hkv, seed=blocks + group, spare_blocks=3))
    announce(f"decode one row of {blocks} blocks, G={group} Hkv={hkv}")
    a, c = run_decode(b, repeat=2)
    compare(a, ref_decode(b), "bf16", f"one row, {blocks} blocks")
    assert np.array_equal(a, c)


@pytest.mark.parametrize("rows", [2, 6, 23, 60])
def test_few_rows_of_all_lengths(rows):
    require_gpu()
    ctx = [int(x) for x in np.exp(np.random.default_rng(rows).uniform(0, np.log(9000), rows))]
    b = W.custom(ctx, [i % 2 for i in range(rows)], 32, 8, seed=rows, spare_blocks=3)
    b.ctx_lens[rows // 2] = 0
    poison_unowned(b)
    announce(f"decode {rows} rows of 1 to 9000 tokens, one empty")
    compare(run_decode(b), ref_decode(b), "bf16", f"{rows} rows")
