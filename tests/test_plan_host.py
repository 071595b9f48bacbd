"""The launch plans' host arithmetic (csrc/plan.h), compiled alone and checked on
the CPU: bounds up to the int32 range's end, every chunk row ranked exactly once,
splits the workspace holds, and limits that follow the compute units."""

import ctypes
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2504_09590_amd", "csrc")
INT32_MAX = 2**31 - 1

WRAPPERS = """
#include "plan.h"
extern "C" {
int longest(int max_ctx, int width) { return bros::longest_blocks(max_ctx, width); }
int items(long long rows, int nkv, int group, int longest, int plan, int resident, int cus) {
  return bros::f32_item_blocks(rows, nkv, group, longest, plan, resident, cus);
}
void chunks(int rows, int seqs, int max_q, int nkv, int pos, int longest, int plan, int cus, long long* out) {
  const bros::F32ChunkPlan p = bros::plan_f32_chunks(rows, seqs, max_q, nkv, pos, longest, plan, cus);
  out[0] = p.units; out[1] = p.tiles_per_seq; out[2] = p.split_blocks; out[3] = p.splits;
}
int whole(long long segments, long long blocks) { return bros::whole_on_any_share(segments, blocks); }
int pieces(long long segments, int group, long long blocks, int cus, long long slots, int* out) {
  return bros::plan_short_decode(segments, group, blocks, cus, slots, out, out + 1);
}
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("plan")
    src, so = d / "plan.cpp", d / "plan.so"
    src.write_text(WRAPPERS)
    subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-ftrapv", "-shared", "-fPIC", "-I", CSRC, str(src),
                    "-o", str(so)], check=True)
    lib = ctypes.CDLL(str(so))
    I, Q = ctypes.c_int, ctypes.c_longlong
    lib.longest.argtypes = [I, I]
    lib.items.argtypes = [Q, I, I, I, I, I, I]
    lib.chunks.argtypes = [I] * 8 + [ctypes.POINTER(Q)]
    lib.whole.argtypes = [Q, Q]
    lib.pieces.argtypes = [Q, I, Q, I, Q, ctypes.POINTER(I)]
    return lib


def plan_blocks(rows, longest):
    """Blocks per split that the fp32 workspace is laid out for (4 to 64, by the rows alone)."""
    sb = 64
    while sb > 4 and rows * -(-longest // sb) < 512:
        sb //= 2
    return sb


def chunk_plan(plan, rows, seqs, max_q, nkv=8, pos=4, longest=100, sb=4, cus=256):
    out = (ctypes.c_longlong * 4)()
    plan.chunks(rows, seqs, max_q, nkv, pos, longest, sb, cus, out)
    return tuple(out)


@pytest.mark.parametrize("max_ctx", [1, 15, 16, 17, INT32_MAX - 15, INT32_MAX - 14, INT32_MAX])
def test_longest_blocks(plan, max_ctx):
    assert plan.longest(max_ctx, INT32_MAX) == max(1, -(-max_ctx // 16))
    assert plan.longest(max_ctx, 7) == min(7, max(1, -(-max_ctx // 16)))
    assert plan.longest(0, 7) == 1


@pytest.mark.parametrize("pos", [16, 8, 4, 2])
def test_loose_row_bounds_plan_as_the_row_count(plan, pos):
    for rows, seqs in ((8, 1), (133, 2), (1279, 256)):
        want = chunk_plan(plan, rows, seqs, rows, pos=pos)
        for max_q in (rows + 1, 1 << 20, INT32_MAX - 1, INT32_MAX):
            assert chunk_plan(plan, rows, seqs, max_q, pos=pos) == want
        assert 0 < want[0] <= 2 * 8 * (rows // pos + seqs)


@pytest.mark.parametrize("pos", [16, 8, 4, 2])
def test_every_tile_has_exactly_one_rank(plan, pos):
    rng = random.Random(pos)
    ranked_by_rows = 0
    for _ in range(300):
        seqs = rng.choice([1, 2, 5, 63, 64, 65, 130])
        longest = rng.choice([1, 3, 40, 700])
        n = [rng.choice([0, 1, 1, 2, rng.randint(0, longest)]) for _ in range(seqs)]
        n[rng.randrange(seqs)] = longest
        cu = [rng.choice([0, 0, 3])]
        for x in n:
            cu.append(cu[-1] + x)
        rows = cu[-1] + rng.choice([0, 0, 5])       # (rows past the last sequence are nobody's)
        units, tiles, _, _ = chunk_plan(plan, rows, seqs, longest, nkv=1, pos=pos)
        seen = []
        for r in range(units):
            if tiles:
                s, t = r % seqs, tiles - 1 - r // seqs
            else:                                   # the last sequence whose first rank is at or before r
                ranked_by_rows += 1
                s = max([i for i in range(seqs) if cu[i] // pos + i <= r], default=0)
                t = cu[s + 1] // pos + s - r
            if 0 <= t and t * pos < n[s]:
                seen.append((s, t))
        assert sorted(seen) == [(s, t) for s in range(seqs) for t in range(-(-n[s] // pos))]
    assert ranked_by_rows > 0


def test_splits_stay_within_the_workspace(plan):
    rng = random.Random(1)
    for _ in range(2000):
        rows, nkv, group = rng.randint(1, 600), rng.choice([1, 3, 8, 64]), rng.choice([1, 2, 4, 8])
        longest = rng.choice([1, 3, 4, 19, 20, 21, 25, 26, rng.randint(1, 3000), 2**27])
        sb = plan_blocks(rows, longest)
        cus = rng.choice([256, 128, 32])
        per = plan.items(rows, nkv, group, longest, sb, 2 * cus, cus)
        assert per % sb == 0 and sb <= per <= 64
        units, tiles, per, splits = chunk_plan(plan, rows, rng.randint(1, rows), rng.randint(1, rows), nkv, 16 // group,
                                               longest, sb, cus)
        assert per % sb == 0 and splits == -(-longest // per) and splits <= -(-longest // sb)


def test_fp32_items(plan):
    # few segments of 8 heads: split (two streams a workgroup walk them); many segments, or a few whose step waits
    # for its host calls: whole
    assert plan.items(1, 1, 8, 20, 4, 512, 256) == 4
    assert plan.items(64, 8, 4, 20, 4, 512, 256) >= 20
    assert plan.items(5, 8, 4, 19, 4, 512, 256) >= 19
    assert plan.items(300, 8, 2, 20, 16, 768, 256) >= 20
    # contexts that may all be near the longest: no more items than run in one round (16 rows of 2048 tokens), and
    # limits that follow the compute units
    assert 16 * 8 * -(-128 // plan.items(16, 8, 8, 128, 4, 512, 256)) <= 512
    assert 4 * 8 * -(-128 // plan.items(4, 8, 8, 128, 4, 128, 64)) <= 128


def short_plan(plan, segments, group, blocks, cus=256, slots=1 << 40):
    out = (ctypes.c_int * 2)()
    return tuple(out) if plan.pieces(segments, group, blocks, cus, slots, out) else None


def test_short_decode_limits_follow_the_compute_units(plan):
    for cus in (256, 128, 64, 32):
        for group in (1, 2, 4, 8):
            for segments in (1, 8, 16, cus // 4, cus // 2 - 1, cus // 2, cus, 2 * cus, 4 * cus, 16 * cus):
                for blocks in list(range(1, 66)) + [94, 200, 511, 1000, 4000]:
                    got = short_plan(plan, segments, group, blocks, cus)
                    # the same segments per compute unit, the same plan
                    if cus != 256 and segments > 16:
                        assert got == short_plan(plan, segments * 256 // cus, group, blocks, 256)
                    if got is not None and got[1] > 1:
                        assert got[1] == -(-blocks // got[0]) <= 64 and segments * got[1] <= 2 * cus
                    if got is not None and got[1] == 1:
                        assert got[0] == blocks <= 64
                    if plan.whole(segments, blocks):       # (decided without the compute units)
                        assert got == (blocks, 1)
    # four rows of 1024 to 4096 tokens, 8 KV heads: pieces of 32 blocks on the whole chip, longer ones on a quarter
    # of it, the even split on an eighth
    assert short_plan(plan, 32, 4, 256) == (32, 8)
    assert short_plan(plan, 32, 4, 256, cus=64) == (64, 4)
    assert short_plan(plan, 32, 4, 256, cus=32) is None


def test_short_decode_partials_fit(plan):
    assert short_plan(plan, 8, 8, 100, slots=8 * 13 * 8) == (8, 13)
    assert short_plan(plan, 8, 8, 100, slots=8 * 13 * 8 - 1) == (16, 7)
    assert short_plan(plan, 2**31, 1, 4) is None and not plan.whole(2**31, 4) and plan.whole(2**31 - 1, 4)
