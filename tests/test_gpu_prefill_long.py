"""bf16 prefill chunks whose context's block table is longer than the LDS copy
holds (more than 32768 positions): the ring variant of the matrix-core kernel.

Whole units (as many units as compute units, so nothing is split) walk the
ring through several refills; with few units the same chunk runs in pieces.
Contexts sit on both sides of a refill boundary, directions per entry, and an
invalid table entry sends all tiles behind it through the masked steps. The
tolerance is the bf16 bar of every other kernel test (the products round P and
the output to bf16 whatever the context's length)."""

import numpy as np
import pytest

import oracle
from paper_2504_09590_amd import workload as W
from tests.gpu_helpers import announce, compare, poison_unowned, require_gpu, with_direction_table
from tests.test_gpu_prefill import chunk_batch, ref_prefill, run_prefill, written

pytestmark = pytest.mark.gpu

RING = 2048 * 16        # positions the LDS copy holds; half of it is refilled at a time


@pytest.mark.parametrize("ctx", [RING + 1, RING + RING // 2 - 16, RING + RING // 2 + 33, 2 * RING + 7])
def test_whole_units_across_refills(ctx):
    require_gpu()
    n = 40
    # 256 one-row chunks beside the long one: more units than a split takes
    b = written(chunk_batch([ctx - n] + [3] * 256, [n] + [1] * 256, [W.RT] * 257, group=4, hkv=1, seed=ctx % 97))
    poison_unowned(b)
    b = with_direction_table(b, seed=5)
    announce(f"prefill ctx {ctx}, whole units, ring refills")
    compare(run_prefill(b), ref_prefill(b), "bf16", f"whole units, ctx {ctx}")


def test_pieces_of_a_long_context():
    require_gpu()
    b = written(chunk_batch([RING + 9000, 100], [70, 33], [W.RT, W.RT], group=8, hkv=2, seed=3))
    poison_unowned(b)
    announce("prefill ctx beyond the LDS table, split")
    compare(run_prefill(b), ref_prefill(b), "bf16", "pieces, long context")


@pytest.mark.parametrize("whole", [True, False])
def test_invalid_entry_early_in_a_long_table(whole):
    # the block behind entry 5 is nobody's: its 16 positions are invisible to every row
    require_gpu()
    n, c0, bad = 33, RING + 20000, 5
    short = 256 if whole else 1
    b = written(chunk_batch([c0] + [3] * short, [n] + [1] * short, [W.RT] * (short + 1), group=4, hkv=1, seed=8))
    poison_unowned(b)
    k = oracle.widen(oracle.gather_kv(b.k_pool, b.block_tables, b.dir, 0, c0 + n), "bf16")
    v = oracle.widen(oracle.gather_kv(b.v_pool, b.block_tables, b.dir, 0, c0 + n), "bf16")
    keep = np.r_[0:16 * bad, 16 * (bad + 1):c0 + n]
    ref = ref_prefill(b)
    ref[:n] = oracle.softmax_attention(oracle.widen(b.q_prefill[:n], "bf16"), k[keep], v[keep],
                                       c0 + 1 + np.arange(n) - 16, oracle.default_scale(b.head_dim))
    b.block_tables[0, bad] = -1
    announce(f"prefill long context, invalid entry {bad}, whole={whole}")
    compare(run_prefill(b), ref, "bf16", "invalid entry, long context")


@pytest.mark.parametrize("whole", [True, False])
def test_long_table_over_a_pool_past_32_bit_offsets(whole):
    # the ring with 64-bit addresses: a pool of more than 2^20 (block, KV head) rows, the batch's blocks behind them
    torch = require_gpu()
    from paper_2504_09590_amd import bros
    n, c0 = 40, RING + RING // 2
    short = 256 if whole else 1
    b = written(chunk_batch([c0] + [3] * short, [n] + [1] * short, [W.RT] * (short + 1), group=4, hkv=2, seed=19))
    poison_unowned(b)
    announce(f"prefill long context, pool rows past 2^20, whole={whole}")
    shift = (1 << 19) + 5                    # x 2 KV heads x 4 KiB: past 4 GiB
    dev = bros.to_device(b)
    big_k = torch.empty((shift + b.num_blocks,) + tuple(dev.k_pool.shape[1:]), dtype=dev.k_pool.dtype, device="cuda")
    big_v = torch.empty_like(big_k)
    big_k[shift:], big_v[shift:] = dev.k_pool, dev.v_pool
    tables = torch.where(dev.block_tables >= 0, dev.block_tables + shift, dev.block_tables)
    P, max_ctx = b.num_prefill, int(b.ctx_lens.max())
    size = bros.bros_attn_workspace_size(1, bros.BROS_BF16, int(b.cu_q[-1]), b.num_q_heads, 128, max_ctx)
    ws = torch.full((size,), 255, dtype=torch.uint8, device="cuda")
    out = torch.full_like(dev.q_prefill, float("nan"))
    bros.bros_attn_prefill_chunk(out, dev.q_prefill, dev.cu_q, n, big_k, big_v, tables[:P].contiguous(), dev.dir[:P],
                                 dev.cls[:P], dev.ctx_lens[:P], max_ctx, workspace=ws)
    torch.cuda.synchronize()
    compare(bros.to_host_bits(out), ref_prefill(b), "bf16", "long table, pool rows past 2^20")
    del big_k, big_v
    torch.cuda.empty_cache()
