"""bf16 decode of short contexts in one launch: contexts and segment counts around
its rule (whole up to 32 blocks with few segments, 32 to 64 by group size and
segments per compute unit with more), all group sizes, empty rows, a max_ctx above every context, invalid table entries and directions
per entry. Against the oracle at the bf16 bar of every other kernel test."""

import numpy as np
import pytest

import oracle
from paper_2504_09590_amd import workload as W
from tests.gpu_helpers import announce, compare, poison_unowned, require_gpu, with_direction_table
from tests.test_gpu_decode import ref_decode, run_decode

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("group,hkv,rows,longest", [
    (1, 8, 5, 512), (2, 3, 5, 513), (4, 8, 7, 512), (8, 1, 3, 17), (4, 8, 8, 1024), (4, 8, 7, 1024), (8, 2, 32, 1024),
    (4, 8, 8, 1025), (2, 1, 200, 700), (4, 8, 300, 90),
    (4, 8, 63, 1024), (4, 8, 64, 769), (4, 8, 65, 768), (2, 8, 64, 512), (2, 8, 65, 513), (1, 8, 65, 384), (1, 8, 65, 385), (8, 8, 65, 1024)])
def test_either_side_of_the_rule(group, hkv, rows, longest):
    require_gpu()
    ctx = [int(x) for x in np.random.default_rng(rows).integers(1, longest + 1, rows)]
    ctx[0] = longest
    b = W.custom(ctx, [i % 2 for i in range(rows)], group * hkv, hkv, seed=rows + longest, spare_blocks=3)
    b.ctx_lens[rows - 1] = 0
    poison_unowned(b)
    b = with_direction_table(b, seed=rows)
    announce(f"decode {rows} rows up to {longest} tokens, G={group} Hkv={hkv}")
    a, c = run_decode(b, repeat=2)
    compare(a, ref_decode(b), "bf16", f"{rows} rows up to {longest}")
    assert np.array_equal(a, c)


@pytest.mark.parametrize("bad", [0, 3, 6])
def test_invalid_entries_are_invisible(bad):
    require_gpu()
    ctx = 16 * 6 + 5
    b = poison_unowned(W.custom([ctx, 40], [W.BE, W.RT], 8, 2, seed=bad, spare_blocks=2))
    k = oracle.widen(oracle.gather_kv(b.k_pool, b.block_tables, b.dir, 0, ctx), "bf16")
    v = oracle.widen(oracle.gather_kv(b.v_pool, b.block_tables, b.dir, 0, ctx), "bf16")
    keep = np.r_[0:16 * bad, min(ctx, 16 * (bad + 1)):ctx]
    ref = ref_decode(b)
    ref[0] = oracle.softmax_attention(oracle.widen(b.q_decode[:1], "bf16"), k[keep], v[keep], np.array([len(keep)]),
                                      oracle.default_scale(128))[0]
    b.block_tables[0, bad] = (-1, b.num_blocks)[bad % 2]
    announce(f"decode with invalid entry {bad}")
    compare(run_decode(b), ref, "bf16", "invalid entry")
