"""bros_kv_gather / bros_kv_scatter at the edges of their workgroups: ids per
workgroup that do and do not divide the list, head counts that are no power of
two, and an id whose rows take several passes. Bytes are exact."""

import numpy as np
import pytest

from tests.gpu_helpers import announce, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("hkv,n", [(1, 127), (1, 129), (3, 42), (3, 43), (8, 16), (8, 17), (8, 1), (7, 100), (200, 3),
                                   (1, 16), (1, 17), (2, 4), (16, 1), (17, 1)])   # (about a chunk per thread)
def test_moves_are_exact(dtype, hkv, n):
    torch = require_gpu()
    from paper_2504_09590_amd import bros
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    blocks = max(4, n // 4)
    g = torch.Generator(device="cuda").manual_seed(n + hkv)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda").to(dt)  # noqa: E731
    k, v, kd, vd = rand(blocks, hkv, 16, 128), rand(blocks, hkv, 16, 128), rand(n, hkv, 128), rand(n, hkv, 128)
    ids = np.random.default_rng(n).permutation(blocks * 16)[:n].astype(np.int32)
    ids[::5] = [(-1, blocks * 16)[i % 2] for i in range(len(ids[::5]))]        # some outside the pool
    inside = torch.from_numpy((ids >= 0) & (ids < blocks * 16)).cuda()
    at = torch.from_numpy(np.clip(ids, 0, blocks * 16 - 1).astype(np.int64)).cuda()
    dev_ids = torch.from_numpy(ids).cuda()
    announce(f"gather and scatter, {n} slots of {hkv} heads, {dtype}")
    ko, vo = torch.full_like(kd, 7), torch.full_like(vd, 7)
    bros.bros_kv_gather(k, v, dev_ids, ko, vo)
    for pool, out in ((k, ko), (v, vo)):
        want = torch.where(inside[:, None, None], pool[at // 16, :, at % 16, :], torch.zeros_like(out))
        assert torch.equal(out, want)
    want = []
    for pool, dense in ((k, kd), (v, vd)):
        w = pool.clone()
        w[at[inside] // 16, :, at[inside] % 16, :] = dense[inside]
        want.append(w)
    bros.bros_kv_scatter(kd, vd, dev_ids, k, v)
    assert torch.equal(k, want[0]) and torch.equal(v, want[1])
