"""max_ctx and max_q_len are upper bounds of a call's lengths: whatever a caller
gives above the true lengths, up to the int32 range's end, every row comes out
as with the tight bounds. Against the oracle at the bar of every other kernel
test of the type."""

import numpy as np
import pytest

from paper_2504_09590_amd import workload as W
from tests.gpu_helpers import announce, compare, poison_unowned, require_gpu
from tests.test_gpu_decode import ref_decode
from tests.test_gpu_prefill import chunk_batch, ref_prefill, written

pytestmark = pytest.mark.gpu

INT32_MAX = 2**31 - 1


def run_with_bounds(batch, max_ctx, max_q=None):
    """The batch's chunks (max_q given) or decode rows under these bounds."""
    import torch
    from paper_2504_09590_amd import bros
    dev = bros.to_device(batch)
    code = bros.BROS_F32 if batch.dtype == "f32" else bros.BROS_BF16
    q = dev.q_decode if max_q is None else dev.q_prefill
    out = torch.full_like(q, float("nan"))
    size = bros.bros_attn_workspace_size(int(max_q is not None), code, q.shape[0], batch.num_q_heads, 128, max_ctx)
    ws = torch.full((size,), 255, dtype=torch.uint8, device="cuda") if size else None
    pools = (dev.k_pool, dev.v_pool, dev.block_tables, dev.dir, dev.cls, dev.ctx_lens, max_ctx)
    if max_q is None:
        bros.bros_attn_decode(out, q, *pools, workspace=ws)
    else:
        bros.bros_attn_prefill_chunk(out, q, dev.cu_q, max_q, *pools, workspace=ws)
    torch.cuda.synchronize()
    return bros.to_host_bits(out)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("group", [1, 8])
@pytest.mark.parametrize("max_ctx", [2100, 40000])
@pytest.mark.parametrize("max_q", [4096, INT32_MAX - 1, INT32_MAX])
def test_chunk_rows_above_the_longest(dtype, group, max_ctx, max_q):
    require_gpu()
    b = poison_unowned(written(chunk_batch([2000, 7], [100, 33], [W.RT, W.BE], group=group, hkv=1, dtype=dtype, seed=group)))
    announce(f"{dtype} chunks G={group} under max_q_len {max_q}, max_ctx {max_ctx}")
    compare(run_with_bounds(b, max_ctx, max_q), ref_prefill(b), dtype, "loose max_q_len")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("max_ctx", [1 << 20, INT32_MAX - 15, INT32_MAX - 14, INT32_MAX])
@pytest.mark.parametrize("chunk", [False, True], ids=["decode", "chunk"])
def test_contexts_above_the_longest(dtype, max_ctx, chunk):
    # contexts of more than one split (64 blocks), which the merge has to fold
    require_gpu()
    if chunk:
        b = written(chunk_batch([2500], [2], [W.RT], group=1, hkv=1, dtype=dtype, seed=3))
    else:
        b = W.custom([2500, 31], [W.RT, W.BE], 1, 1, dtype=dtype, seed=3, spare_blocks=3)
    poison_unowned(b)
    announce(f"{dtype} {'chunk' if chunk else 'decode'} under max_ctx {max_ctx}")
    ref = ref_prefill(b) if chunk else ref_decode(b)
    compare(run_with_bounds(b, max_ctx, 2 if chunk else None), ref, dtype, "loose max_ctx")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rows,c0", [([8], 4000), ([8] * 16, 1000), ([200] + [1] * 31, 300)])
def test_a_loose_row_bound_changes_no_bit(dtype, rows, c0):
    # the same units, split the same way: the rows say how far they can be split, not the bound
    require_gpu()
    b = written(chunk_batch([c0] * len(rows), rows, [W.RT] * len(rows), group=4, hkv=2, dtype=dtype, seed=len(rows)))
    poison_unowned(b)
    announce(f"{dtype} chunks of {rows[:2]}... rows under loose max_q_len")
    tight = run_with_bounds(b, c0 + max(rows), sum(rows))
    compare(tight, ref_prefill(b), dtype, "the row count as bound")
    for max_q in (8192, INT32_MAX):
        assert np.array_equal(tight, run_with_bounds(b, c0 + max(rows), max_q))
