"""Split units of the bf16 prefill: the piece plan on both sides of 64 items
(up to 64 every wave plans by itself, beyond the workgroup does in LDS), items
without rows among them, ranks past the pieces, and a workspace that holds few
partials. The tolerance is the bf16 bar of every other kernel test."""

import numpy as np
import pytest

import oracle
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


@pytest.mark.parametrize("group,hkv,n,c0", [(1, 16, 1500, 1900), (8, 1, 1100, 2500), (8, 1, 3300, 0), (2, 8, 1500, 3000)])
def test_units_cut_into_two_pieces_per_compute_unit(group, hkv, n, c0):
    # nearly as many units as compute units: one piece each would leave the longest ones whole
    require_gpu()
    b = written(chunk_batch([c0], [n], [W.RT], group=group, hkv=hkv, seed=n))
    poison_unowned(b)
    announce(f"prefill {n} rows on {c0} tokens, G={group} Hkv={hkv}, two pieces per compute unit")
    got = run_prefill(b)
    rows = np.r_[0:40, n // 2:n // 2 + 20, n - 40:n]      # (the oracle on some of the rows)
    k = oracle.widen(oracle.gather_kv(b.k_pool, b.block_tables, b.dir, 0, c0 + n), "bf16")
    v = oracle.widen(oracle.gather_kv(b.v_pool, b.block_tables, b.dir, 0, c0 + n), "bf16")
    ref = oracle.softmax_attention(oracle.widen(b.q_prefill[rows], "bf16"), k, v, c0 + 1 + rows, oracle.default_scale(128))
    compare(got[rows], ref, "bf16", "two pieces per compute unit")
    assert np.isfinite(oracle.widen(got, "bf16")).all()


def test_part_sizes_of_nearly_as_many_units_as_compute_units():
    # 192 units of 192 to 284 key tiles on 256 compute units. One piece per compute unit means that most
    # stay whole, 155 us; cut into two and three pieces each 111. The list of split units lies behind the
    # partials (1024 of 128 rows of 130 floats): count, then (item, parts, first slot).
    torch = require_gpu()
    from paper_2504_09590_amd import bros
    b = chunk_batch([6000], [3072], [W.RT], group=1, hkv=8, seed=1)
    dev = bros.to_device(b)
    size = bros.bros_attn_workspace_size(1, bros.BROS_BF16, 3072, 8, 128, 9072)
    ws = torch.zeros(size, dtype=torch.uint8, device="cuda")
    out = torch.empty_like(dev.q_prefill)
    announce("prefill part sizes, 192 units")
    bros.bros_attn_prefill_chunk(out, dev.q_prefill, dev.cu_q, 3072, dev.k_pool, dev.v_pool, dev.block_tables[:1],
                                 dev.dir[:1], dev.cls[:1], dev.ctx_lens[:1], 9072, workspace=ws)
    torch.cuda.synchronize()
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the figures are for 256 compute units")
    split = ws.cpu().numpy().view(np.int32)[1024 * 128 * 130:]
    parts = {int(i): int(p) for i, p, _ in split[1:1 + 3 * split[0]].reshape(-1, 3)}
    tiles = [-(-(6000 + 128 * (t + 1)) // 32) for t in range(24)]
    pieces = [-(-tiles[t] // parts.get(t, 1)) for t in range(24)]
    assert max(pieces) <= 150 and sum(parts.get(t, 1) for t in range(24)) <= 64
