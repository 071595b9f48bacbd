"""Split units of the bf16 prefill: the piece plan on both sides of 64 items
(up to 64 every wave plans by itself, beyond the workgroup does in LDS), items
without rows among them, ranks past the pieces, and a workspace that holds few
partials. The tolerance is the bf16 bar of every other kernel test."""

import numpy as np
import pytest

from paper_2504_09590_amd import workload as W
from tests.gpu_helpers import announce, compare, poison_unowned, require_gpu
from tests.test_gpu_prefill import chunk_batch, ref_prefill, run_prefill, written

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("items", [2, 63, 64, 65, 200])
def test_plan_either_side_of_a_wave(items):
    require_gpu()
    c0 = [12000, 3000] + [int(x) for x in np.random.default_rng(items).integers(0, 40, items - 2)]
    n = [32, 20] + [(i * 7) % 33 for i in range(items - 2)]      # some without rows
    b = written(chunk_batch(c0, n, [W.RT] * items, group=4, hkv=1, seed=items))
    poison_unowned(b)
    announce(f"prefill split plan, {items} items")
    split, whole = run_prefill(b), run_prefill(b, workspace=False)
    ref = ref_prefill(b)
    compare(split, ref, "bf16", f"split, {items} items")
    compare(whole, ref, "bf16", f"whole, {items} items")
    assert not np.array_equal(split, whole)


@pytest.mark.parametrize("c0,n", [(16 * 94, 32), (16 * 96 - 1, 33), (700, 300), (1100, 129)])
def test_units_around_the_split_rule(c0, n):
    require_gpu()
    b = written(chunk_batch([c0, 0], [n, 17], [W.RT, W.RT], group=4, hkv=8, seed=n))
    poison_unowned(b)
    announce(f"prefill c0={c0} n={n} near the split rule")
    compare(run_prefill(b), ref_prefill(b), "bf16", "near the split rule")


def test_long_context_with_room_for_few_partials():
    # beyond 32768 positions the workspace may hold only a few partials: 8 heads
    # x 4 row tiles share what the query's size gives
    require_gpu()
    b = written(chunk_batch([33000], [100], [W.RT], group=1, hkv=8, seed=4))
    poison_unowned(b)
    announce("prefill beyond the LDS table with a small workspace")
    compare(run_prefill(b), ref_prefill(b), "bf16", "few partials")
