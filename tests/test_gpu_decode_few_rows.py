"""bf16 decode of few rows: contexts in pieces of 8, 16, 32 or 64 blocks, one
workgroup each, and their merge (a round per eight partials); beyond 64 pieces
the even split, whose merge's waves share a segment's many partials, and which
gives a wave up to four tiles when one long context stands among short ones.
Against the oracle at the bf16 bar of every other kernel test, and twice
bitwise."""

import numpy as np
import pytest

import oracle
from paper_2504_09590_amd import workload as W
from tests.gpu_helpers import announce, compare, poison_unowned, require_gpu
from tests.test_gpu_decode import ref_decode, run_decode

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("group,hkv", [(1, 8), (2, 2), (4, 8), (8, 1)])
# whole; then 5 pieces of 8 blocks, 16 and 17 (two rounds and three), and pieces of 16 and 32 blocks
@pytest.mark.parametrize("blocks", [1, 32, 33, 128, 129, 1000, 1024, 1025])
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


@pytest.mark.parametrize("group", [1, 8])
def test_even_split_of_one_very_long_row(group):
    # more than 64 pieces of 64 blocks: the even split, a thousand partials in one segment
    require_gpu()
    b = W.custom([16 * 4100 - 3, 30], [W.BE, W.RT], group, 1, seed=group, spare_blocks=3)
    poison_unowned(b)
    announce(f"decode one row of 4100 blocks, G={group}")
    compare(run_decode(b), ref_decode(b), "bf16", "4100 blocks")


def test_one_long_row_among_many_short_ones():
    # the longest context alone sets the pieces: too many of them, and few tiles for the even split
    require_gpu()
    ctx = [5, 9000] + [int(x) for x in np.random.default_rng(7).integers(1, 60, 98)]
    b = poison_unowned(W.custom(ctx, [i % 2 for i in range(100)], 32, 8, seed=7, spare_blocks=3))
    announce("decode one long row among 99 short ones")
    compare(run_decode(b), ref_decode(b), "bf16", "one long row among short ones")


@pytest.mark.parametrize("ctx,pos", [([1], 0), ([300], 299), ([300, 40], 17), ([9000], 4321)])
@pytest.mark.parametrize("value", [np.inf, -np.inf])
def test_infinite_values_stay_infinite(ctx, pos, value):
    # a V value of infinity, under weights of 1 (a lone token) and less: the result's dim is that infinity, not a NaN
    require_gpu()
    b = W.custom(ctx, [i % 2 for i in range(len(ctx))], 8, 2, seed=pos, spare_blocks=3)
    blk, slot = oracle.physical_location(b.block_tables, b.dir, 0, np.array([pos]))
    ref = ref_decode(b)
    b.v_pool[blk[0], :, slot[0], 5] = np.uint16(0x7F80 if value > 0 else 0xFF80)
    announce(f"decode of contexts {ctx}, a V value of {value} at {pos}")
    got = oracle.widen(run_decode(b), "bf16")
    assert (got[0, :, 5] == value).all()
    ref[0, :, 5] = got[0, :, 5] = 0.0
    assert np.isfinite(got).all() and np.abs(got - ref).max() <= 2e-2


# pieces that do not fill a round of eight of the merge: 3, 36 (twice) and 9 of 16 blocks
@pytest.mark.parametrize("ctx,pos", [([600], 599), ([9000], 8999), ([9000, 40], 8960), ([2300, 2048], 2299)])
@pytest.mark.parametrize("value", [np.inf, -np.inf])
def test_infinite_values_of_the_last_piece(ctx, pos, value):
    require_gpu()
    b = W.custom(ctx, [i % 2 for i in range(len(ctx))], 8, 2, seed=pos, spare_blocks=3)
    blk, slot = oracle.physical_location(b.block_tables, b.dir, 0, np.array([pos]))
    ref = ref_decode(b)
    b.v_pool[blk[0], :, slot[0], 5] = np.uint16(0x7F80 if value > 0 else 0xFF80)
    announce(f"decode of contexts {ctx}, a V value of {value} at {pos}, in the last piece")
    got = oracle.widen(run_decode(b), "bf16")
    assert (got[0, :, 5] == value).all()
    ref[0, :, 5] = got[0, :, 5] = 0.0
    assert np.isfinite(got).all() and np.abs(got - ref).max() <= 2e-2


# the edges of the pieces: whole up to 32 blocks, 8 blocks (up to 24 pieces), 16, 32 and 64 (up to 64 pieces), each
# only while the pieces of all rows are few
@pytest.mark.parametrize("group,hkv,rows", [(1, 2, 1), (8, 1, 1), (4, 8, 1), (4, 17, 1), (8, 2, 9)])
@pytest.mark.parametrize("blocks", [32, 33, 192, 193, 1024, 1025, 2048, 2049])
def test_edges_of_the_pieces(group, hkv, rows, blocks):
    require_gpu()
    ctx = [16 * blocks - (blocks % 5)] + [17 * i + 3 for i in range(1, rows)]
    b = poison_unowned(W.custom(ctx, [i % 2 for i in range(rows)], group * hkv, hkv, seed=blocks + group, spare_blocks=3))
    announce(f"decode {rows} rows, the longest of {blocks} blocks, G={group} Hkv={hkv}")
    compare(run_decode(b), ref_decode(b), "bf16", f"{blocks} blocks")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("cus", [64, 32])
def test_decode_on_a_compute_unit_share(dtype, cus):
    # its limits follow the share's compute units: other pieces, or the even split, than on the whole chip
    torch = require_gpu()
    from paper_2504_09590_amd import bros
    code = bros.BROS_F32 if dtype == "f32" else bros.BROS_BF16
    share = bros.bros_stream_create_cu_share(0, cus)
    try:
        for ctx in ([1300, 4000, 2047, 2999], [400] * 20 + [17], [900], [60] * 40):
            b = poison_unowned(W.custom(ctx, [i % 2 for i in range(len(ctx))], 16, 8, dtype=dtype, seed=len(ctx),
                                        spare_blocks=3))
            announce(f"{dtype} decode of {len(ctx)} rows on {cus} compute units")
            dev = bros.to_device(b)
            out = torch.full_like(dev.q_decode, float("nan"))
            size = bros.bros_attn_workspace_size(0, code, len(ctx), 16, 128, max(ctx))
            ws = torch.full((max(size, 16),), 255, dtype=torch.uint8, device="cuda")
            torch.cuda.synchronize()
            bros.bros_attn_decode(out, dev.q_decode, dev.k_pool, dev.v_pool, dev.block_tables, dev.dir, dev.cls,
                                  dev.ctx_lens, max(ctx), workspace=ws, stream=share)
            torch.cuda.synchronize()
            compare(bros.to_host_bits(out), ref_decode(b), dtype, f"{len(ctx)} rows on a share")
    finally:
        torch.cuda.synchronize()
        bros.bros_stream_destroy(share)
