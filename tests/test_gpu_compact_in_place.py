"""Compaction into the lists' own memory: the records over the pool, at the same
place or shifted, or the table over it; bricks of every size class, 32- and
64-bit keys. The result is that of separate memory, bit for bit."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2211_15460_amd import scenes as S
from tests.gpu_util import u32, u64
from tests.test_gpu_bricks import F, check, expected, records  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("where", ["frag", "frag_after", "frag_before", "table"])
@pytest.mark.parametrize("sizes", [(1,), (200, 256, 257, 64), (1024, 1025, 3, 8192, 8193, 20000)])
def test_outputs_over_the_pool(F, sizes, where):  # noqa: F811
    import torch
    g = np.random.default_rng(len(sizes))
    bricks = np.sort(g.choice(64, len(sizes), replace=False))   # of depth 5
    keys = np.concatenate([b * 512 + g.integers(0, 512, n) for b, n in zip(bricks, sizes)])
    keys = keys[g.permutation(keys.size)]
    recs = records(g, keys.size, 50)
    n, cap = keys.size, keys.size + 37
    d = F.desc(F.FHV_POFL, levels=5)
    lists = F.alloc_lists(d, cap)
    shift = cap // 2 + 1
    room = torch.empty((cap + 2 * shift, 4), dtype=torch.int32, device="cuda")
    lists.pool = room[shift:shift + cap]
    lists.pool[:n] = torch.from_numpy(recs.view(np.int32)).cuda()
    lists.keys[:n] = torch.from_numpy(keys.astype(np.uint32).view(np.int32)).cuda()
    lists.counter.fill_(n)
    out = F.alloc_pofa(cap)
    if where == "table":   # 8 + 4 + 4 bytes a row: the pool's own 16 a slot
        flat = lists.pool.reshape(-1)
        out.oct_key = flat[:2 * cap].view(torch.int64)
        out.oct_off, out.oct_cnt = flat[2 * cap:3 * cap], flat[3 * cap:]
    else:
        at = {"frag": shift, "frag_after": 2 * shift, "frag_before": 0}[where]
        out.frag = room[at:at + cap]
    F.compact(lists, d, out)
    torch.cuda.synchronize()
    k = int(out.n_occ.item())
    check({"key": u64(out.oct_key)[:k], "off": u32(out.oct_off)[:k], "cnt": u32(out.oct_cnt)[:k],
           "frag": u32(out.frag)[:n], "n_occ": k, "n_frag": int(out.n_frag.item())}, expected(keys, recs))


def test_batch_of_64_bit_keys(F):  # noqa: F811
    """A batch whose key space is beyond 2^32, its arrays over its pool."""
    import torch
    L, n = 9, 33
    b = F.to_device_batch([S.cube_scene(60, 40 + i, scale_range=(0.02, 0.05), ground=0) for i in range(n)], L)
    vm = F.batch_view_matrices([[S.cube_view(0.0, L, 16, 16)]] * n)
    img = F.alloc_images(n, 16, 16)
    first = F.alloc_batch_lists(b, 0)
    F.batch_run(b, vm, 16, 16, 1, first, F.alloc_pofa(0), img)
    cap = int(first.counter.item())
    assert cap > 0
    got = []
    for in_place in (False, True):
        lists, out = F.alloc_batch_lists(b, cap), F.alloc_pofa(cap)
        assert lists.keys.dtype == torch.int64
        if in_place:
            out.frag = lists.pool
        F.batch_run(b, vm, 16, 16, 1, lists, out, img)
        k = int(out.n_occ.item())
        got.append([out.oct_key[:k].clone(), out.oct_off[:k].clone(), out.oct_cnt[:k].clone(), out.frag.clone(),
                    img.zbuf.clone(), img.rgba.clone(), out.n_frag.clone()])
    for x, y in zip(*got):
        assert torch.equal(x, y)
