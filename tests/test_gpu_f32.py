"""fp32 chunks on the matrix instructions, and fp32 decode rows: the edges of the
16-slot blocks, of the four waves that share a unit, of splits over workgroups
and of units of 16 / G positions, all group sizes, both directions, and
non-finite V rows that only later rows see. Against the oracle at the fp32 bar
of every other kernel test (1e-5)."""

import numpy as np
import pytest

import oracle
from paper_2504_09590_amd import workload as W
from tests.gpu_helpers import announce, compare, poison_unowned, require_gpu, with_direction_table
from tests.test_gpu_decode import ref_decode, run_decode
from tests.test_gpu_prefill import chunk_batch, ref_prefill, run_prefill, written

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("group,hkv", [(1, 8), (2, 3), (4, 2), (8, 1)])
def test_chunks_all_groups_ragged(group, hkv):
    require_gpu()
    b = written(chunk_batch([0, 1, 15, 16, 700, 0], [1, 17, 33, 100, 65, 0], [W.RT, W.BE] * 3, group=group, hkv=hkv,
                            dtype="f32", seed=40 + group))
    poison_unowned(b)
    b = with_direction_table(b, seed=group)
    announce(f"f32 chunks G={group} Hkv={hkv}")
    compare(run_prefill(b), ref_prefill(b), "f32", f"f32 chunks G={group}")


@pytest.mark.parametrize("c0,n", [(4000, 1), (4090, 7), (1023, 2), (511, 16), (16 * 64 - 5, 9)])
def test_few_rows_on_a_long_context_split(c0, n):
    # few units: their blocks go to several workgroups, and rows of one unit may need different numbers of splits
    require_gpu()
    b = written(chunk_batch([c0], [n], [W.RT], group=2, hkv=2, dtype="f32", seed=n))
    poison_unowned(b)
    announce(f"f32 chunk c0={c0} n={n}, split")
    compare(run_prefill(b), ref_prefill(b), "f32", f"f32 c0={c0} n={n}")


@pytest.mark.parametrize("group", [1, 4, 8])
@pytest.mark.parametrize("rows", [1, 5, 300])
def test_decode_rows_split_and_whole(group, rows):
    require_gpu()
    rng = np.random.default_rng(rows)
    ctx = [int(x) for x in rng.integers(1, 5000 if rows < 10 else 200, rows)]
    ctx[0] = 5000 if rows < 10 else 128       # the longest fills whole blocks
    b = W.custom(ctx, [i % 2 for i in range(rows)], 2 * group, 2, dtype="f32", seed=rows + group, spare_blocks=3)
    if rows == 300:
        b.ctx_lens[7] = 0                     # a row without context is zeros
    poison_unowned(b)
    announce(f"f32 decode rows={rows} G={group}")
    compare(run_decode(b), ref_decode(b), "f32", f"f32 decode rows={rows} G={group}")


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_non_finite_values_of_later_positions(value):
    # position 37 holds a non-finite V row: rows before it must not notice, whatever shares their unit
    require_gpu()
    b = written(chunk_batch([20], [40], [W.RT], group=2, hkv=2, dtype="f32", seed=9))
    blk, slot = oracle.physical_location(b.block_tables, b.dir, 0, np.array([37]))
    ref = ref_prefill(b)
    b.v_pool[blk[0], :, slot[0], 5] = value
    announce(f"f32 chunk with a V row of {value}")
    got = run_prefill(b)
    before = 37 - 20
    compare(got[:before], ref[:before], "f32", "rows before the non-finite position")
    assert not np.isfinite(got[before:, :, 5]).any()
    rest = [d for d in range(128) if d != 5]
    compare(got[before:][:, :, rest], ref[before:][:, :, rest], "f32", "other dims")


@pytest.mark.parametrize("group,hkv", [(1, 3), (4, 2), (8, 1)])
@pytest.mark.parametrize("c0", [0, 1500])
def test_one_long_chunk_among_short_ones(group, hkv, c0):
    # ranked by their rows: over 64 sequences (a second step of the search), empty ones, a last one of several tiles
    require_gpu()
    n = [1] * 66 + [0, 130, 0, 0] + [1, 2, 0] * 5 + [35]
    b = written(chunk_batch([c0 if x > 1 else 7 for x in n], n, [W.RT, W.BE] * (len(n) // 2), group=group, hkv=hkv,
                            dtype="f32", seed=group + c0))
    poison_unowned(b)
    announce(f"f32 chunks, one of 130 rows among short ones, G={group} c0={c0}")
    compare(run_prefill(b), ref_prefill(b), "f32", "one long chunk among short ones")


# one item per context, and items of 4 to 32 blocks; beyond the plan's blocks each block is summed by itself
@pytest.mark.parametrize("group,hkv,rows,longest", [
    (1, 8, 4, 320), (8, 1, 1, 320), (4, 8, 64, 320), (2, 8, 12, 512), (4, 8, 16, 2048), (2, 8, 128, 400), (4, 2, 130, 417),
    (8, 2, 40, 1000)])
def test_decode_item_sizes(group, hkv, rows, longest):
    require_gpu()
    ctx = [int(x) for x in np.random.default_rng(rows).integers(1, longest + 1, rows)]
    ctx[0] = longest
    b = W.custom(ctx, [i % 2 for i in range(rows)], group * hkv, hkv, dtype="f32", seed=rows + longest, spare_blocks=3)
    poison_unowned(b)
    announce(f"f32 decode {rows} rows up to {longest} tokens, G={group} Hkv={hkv}")
    compare(run_decode(b), ref_decode(b), "f32", f"f32 {rows} rows up to {longest}")


# Distance from 64 bits (2-norm over the result's) of these batches with items of the plan's length, 4
# blocks and a partial each, which is the bound. Longer items summed in one chain were at 1.432e-7,
# 1.688e-7 and 1.854e-7, block by block they are at 1.333e-7, 1.543e-7 and 1.613e-7.
@pytest.mark.parametrize("group,hkv,rows,lo,hi,bound", [
    (1, 8, 64, 17, 300, 1.400e-7), (4, 8, 16, 64, 2048, 1.667e-7), (2, 8, 40, 300, 1384, 1.689e-7)])
def test_longer_items_keep_the_precision(group, hkv, rows, lo, hi, bound):
    require_gpu()
    ctx = [int(x) for x in np.random.default_rng(rows).integers(lo, hi + 1, rows)]
    b = W.custom(ctx, [W.BE] * rows, group * hkv, hkv, dtype="f32", seed=rows, spare_blocks=3)
    announce(f"f32 decode {rows} rows of {lo} to {hi} tokens, distance from 64 bits")
    ref = ref_decode(b)
    err = float(np.linalg.norm(run_decode(b) - ref) / np.linalg.norm(ref))
    print(f"distance {err:.4g}")
    assert err <= bound


@pytest.mark.parametrize("bad", [0, 3, 60, 94])
@pytest.mark.parametrize("c0,n", [(1490, 25), (1510, 1)])
def test_chunk_entries_out_of_range_are_invisible(bad, c0, n):
    # the first, a middle and the tail block of whole units and of split ones; block 0, read in place
    # of an invalid entry's, holds NaNs
    require_gpu()
    for units in (1, 80):                     # alone its blocks are split, among 80 others not
        b = written(chunk_batch([c0] + [3] * (units - 1), [n] + [20] * (units - 1), [W.RT] * units, group=4, hkv=2,
                                dtype="f32", seed=bad))
        b = poison_unowned(b)
        tab = b.block_tables
        spare = np.setdiff1d(np.arange(b.num_blocks), tab[tab >= 0])[0]
        if 0 in tab:                          # another block takes the place of block 0
            b.k_pool[spare], b.v_pool[spare] = b.k_pool[0], b.v_pool[0]
            tab[tab == 0] = spare
        b.k_pool[0] = b.v_pool[0] = np.nan
        k = oracle.gather_kv(b.k_pool, tab, b.dir, 0, c0 + n)
        v = oracle.gather_kv(b.v_pool, tab, b.dir, 0, c0 + n)
        ref = ref_prefill(b)
        gone = np.arange(16 * bad, min(16 * (bad + 1), c0 + n))
        for j in range(n):
            keep = np.setdiff1d(np.arange(c0 + j + 1), gone)
            ref[j] = oracle.softmax_attention(b.q_prefill[j:j + 1].astype(np.float64), k[keep].astype(np.float64),
                                              v[keep].astype(np.float64), np.array([len(keep)]),
                                              oracle.default_scale(128))[0]
        for entry in (-1, b.num_blocks):
            tab[0, bad] = entry
            announce(f"f32 chunk of {n} rows, entry {bad} is {entry}, {units} units")
            compare(run_prefill(b), ref, "f32", f"invalid entry {bad}")
