"""Capture of triangles on both sides of every bound at which the rasterizer
changes its arithmetic: boxes of 2^30 square fixed-point units and of 2^22
units a side (linear forms in 32-bit edges and doubles against 64-bit
integers), twice the area of 2^26 units (depth by remainder), one tile and
many tiles per triangle. Lists equal the oracle's fragment by fragment."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2211_15460_amd import scenes as S
from tests.gpu_util import run_capture
from tests.listutil import canonical, walk_lists

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2211_15460_amd import fhv
    fhv.lib()
    return fhv


def sized_soup(n, seed, sizes, lo, hi):
    """n triangles with random corners in boxes whose sides (in units of the
    cube [lo, hi]) are drawn from `sizes`, one corner pair spanning the box;
    random colours of all four bytes, random object bytes."""
    g = np.random.default_rng(seed)
    side = g.choice(sizes, (n, 1, 1)) * np.ones((1, 1, 3))
    base = g.random((n, 1, 3)) * (1.0 - side)
    c = g.random((n, 3, 3))
    c[:, 0], c[:, 1, :2] = 0.0, 1.0
    p = lo + (hi - lo) * np.clip(base + side * c, 0.0, 1.0 - 2.0 ** -20)
    nv = 3 * n
    return S.Mesh(p.reshape(nv, 3).astype(np.float32), g.integers(0, 2 ** 32, nv, dtype=np.uint32),
                  np.arange(nv, dtype=np.uint32).reshape(n, 3), g.integers(0, 256, n).astype(np.uint8))


def compare(F, mesh, d, o):
    o_head, o_pool, o_cnt = o
    cap = max(int(o_cnt), 1)
    head, pool, keys, cnt, _ = run_capture(F, mesh, d, cap)
    print(f"fragments {cnt}", flush=True)
    assert cnt == o_cnt
    assert np.array_equal(canonical(*walk_lists(head, pool, cnt)), canonical(*walk_lists(o_head, o_pool, o_cnt)))


# sizes in pixels of the window's longer side; 32 pixels a side is an area of
# 2^26 units, 128 a box of 2^30
@pytest.mark.parametrize("W,H,n,pixels", [(512, 512, 400, (1, 5, 9, 30, 32, 33)), (512, 512, 60, (127, 128, 129, 200)),
                                          (1000, 700, 8, (600, 1000)), (16384, 5, 12, (16000, 16384)),
                                          (7, 9000, 12, (8000, 9000))])
def test_pixel_capture_forms(F, orc, W, H, n, pixels):
    mesh = sized_soup(n, W + n, np.array(pixels) / max(W, H), -1.0, 1.0)
    cap = 1 << 21
    compare(F, mesh, F.desc(F.FHV_PPFL, W, H), orc.capture_ppfl(mesh, W, H, cap))


# sizes in samples (2^(L+1) per cube side)
@pytest.mark.parametrize("L,n,samples", [(7, 200, (1, 7, 8, 9, 40)), (8, 30, (80, 90, 128, 129)), (8, 6, (300, 500))])
@pytest.mark.parametrize("proj", [0, 3])
def test_octant_capture_forms(F, orc, L, n, samples, proj):
    mesh = sized_soup(n, L + n, np.array(samples) / 2.0 ** (L + 1), 0.0, 1.0)
    compare(F, mesh, F.desc(F.FHV_POFL, levels=L, projection=proj), orc.capture_pofl(mesh, L, 1 << 22, projection=proj))
