"""Compaction at the sizes where it changes its way: bricks (512 consecutive
keys) of up to 256, 1,024 and 8,192 records and beyond, few and many bricks,
bricks whose numbers share their low bits, runs of equal records; and arrays
straight from dense scenes. Against numpy's stable sort and the oracle."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2211_15460_amd import scenes as S
from tests.gpu_util import run_capture, run_compact, u32, u64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2211_15460_amd import fhv
    fhv.lib()
    return fhv


def compact_of(F, keys, recs, levels, capacity):
    """fhv_compact of a pool holding these keys and records in this order."""
    import torch
    n = keys.size
    d = F.desc(F.FHV_POFL, levels=levels)
    lists = F.alloc_lists(d, capacity)
    lists.pool[:n] = torch.from_numpy(recs.view(np.int32)).cuda()
    lists.keys[:n] = torch.from_numpy(keys.astype(np.uint32).view(np.int32)).cuda()
    lists.counter.fill_(n)
    return run_compact(F, lists, d)[0]


def expected(keys, recs):
    order = np.lexsort((recs[:, 2], recs[:, 1], recs[:, 0], keys))
    k, r = keys[order], recs[order].copy()
    table, first, count = np.unique(k, return_index=True, return_counts=True)
    r[:, 3] = np.repeat(np.arange(table.size, dtype=np.uint32), count)
    return {"key": table.astype(np.uint64), "off": first.astype(np.uint32), "cnt": count.astype(np.uint32), "frag": r}


def check(got, want):
    assert got["n_occ"] == want["key"].size and got["n_frag"] == want["frag"].shape[0]
    for f in ("key", "off", "cnt", "frag"):
        assert np.array_equal(got[f], want[f]), f


def records(g, n, few):
    """n records; `few` distinct values per word, so that many tie."""
    return g.integers(0, few, (n, 4), dtype=np.uint32)


@pytest.mark.parametrize("sizes", [(1,), (63, 64, 65), (255, 256, 257), (1, 1023, 1024, 1025, 2), (8191, 8192, 8193),
                                   (30000, 5, 300), (70000,)])
@pytest.mark.parametrize("few", [3, 2 ** 32 - 1])
def test_brick_sizes(F, sizes, few):
    g = np.random.default_rng(sum(sizes))
    bricks = np.sort(g.choice(64, len(sizes), replace=False))   # of depth 5
    keys = np.concatenate([b * 512 + g.integers(0, 512, n) for b, n in zip(bricks, sizes)])
    keys = keys[g.permutation(keys.size)]
    recs = records(g, keys.size, few)
    check(compact_of(F, keys, recs, 5, keys.size), expected(keys, recs))


@pytest.mark.parametrize("n,n_bricks,step", [(20000, 40, 1), (20000, 40, 512), (40000, 3000, 1), (2047, 700, 16),
                                             (2049, 32768, 1)])
def test_brick_numbers(F, n, n_bricks, step):
    """Consecutive bricks, bricks 512 apart (equal low bits) and more bricks
    than a workgroup's counters, in a pool with room to spare."""
    g = np.random.default_rng(n + step)
    keys = (g.integers(0, n_bricks, n) * step % 32768) * 512 + g.integers(0, 512, n)
    recs = records(g, n, 1000)
    check(compact_of(F, keys, recs, 8, n + 5000), expected(keys, recs))


@pytest.mark.parametrize("L,n_tri", [(3, 200), (4, 300), (5, 300)])
def test_dense_arrays(F, orc, L, n_tri):
    """Few octants with many fragments: both ways to arrays, the oracle's
    compaction of its own lists as the result."""
    g = np.random.default_rng(L)
    nv = 3 * n_tri
    mesh = S.Mesh(g.random((nv, 3)).astype(np.float32), g.integers(0, 2 ** 32, nv, dtype=np.uint32),
                  np.arange(nv, dtype=np.uint32).reshape(n_tri, 3), g.integers(0, 256, n_tri).astype(np.uint8))
    d = F.desc(F.FHV_POFL, levels=L)
    want = orc.compact(*orc.capture_pofl(mesh, L, 1 << 20))
    n, n_occ = want["frag"].shape[0], want["n_occ"]
    *_, lists = run_capture(F, mesh, d, n + 100)
    check(run_compact(F, lists, d)[0], want)
    out = F.capture_arrays(F.to_device(mesh), d, F.alloc_pofa(n + 100))
    assert int(out.n_frag.item()) == n and int(out.n_occ.item()) == n_occ
    assert np.array_equal(u32(out.frag)[:n], want["frag"])
    assert np.array_equal(u64(out.oct_key)[:n_occ], want["key"])
    assert np.array_equal(u32(out.oct_off)[:n_occ], want["off"])
    assert np.array_equal(u32(out.oct_cnt)[:n_occ], want["cnt"])
    # arrays too small for the scene (and for its occupied bricks): the count alone
    small = F.capture_arrays(F.to_device(mesh), d, F.alloc_pofa(1))
    assert int(small.n_frag.item()) == n and int(small.n_occ.item()) == 0
