"""Transparent rays at depths of every scale, against the oracle bit for bit: a
viewer inside the scene (depths from next to zero up), depths in grid units and
at either end of float, with more hits in a tile than a slab holds, so that the
slabs' keys run over many binary orders; depths that overflow. By the tiles and,
where their boxes do not fit, by the octree walk."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2211_15460_amd import scenes as S
from tests.test_gpu_ray_tiles import F, both, compare, fits  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def squares(items, alpha, seed):
    """Squares facing the z axis, (x, y, z, side) each, random colours."""
    rng = np.random.default_rng(seed)
    pos, col = [], []
    for x, y, z, s in items:
        c = int(rng.integers(0, 1 << 24)) | (alpha << 24)
        for tri in (((x, y, z), (x + s, y, z), (x + s, y + s, z)), ((x, y, z), (x + s, y + s, z), (x, y + s, z))):
            pos.extend(tri)
            col.extend([c] * 3)
    pos = np.asarray(pos, np.float32)
    return S.Mesh(pos, np.asarray(col, np.uint32), np.arange(pos.shape[0], dtype=np.uint32).reshape(-1, 3),
                  np.zeros(pos.shape[0] // 3, np.uint8))


def depth_view(theta, L, W, H, unit, at):
    """An orbit view whose depths are `unit` per grid unit, zero at the scene
    point `at`."""
    v = S.cube_view(theta, L, W, H, splat_px=1)
    m = v.m.astype(np.float64)
    m[2] *= unit / np.linalg.norm(m[2, :3])
    m[2, 3] = -(m[2, :3] @ (np.asarray(at) * 2.0 ** (L + 8)))
    return S.View(m.astype(np.float32), W, H, 1)


def near_and_far(bulk, near_z=0.02):
    """A few samples of small squares next to the viewer in every tile, and
    `bulk` large ones far behind them."""
    near = [(0.2 + 0.07 * i, 0.2 + 0.07 * j, near_z, 0.008) for i in range(9) for j in range(9)]
    return squares(near + [(0.1, 0.1, 0.9 + 0.02 * k, 0.8) for k in range(bulk)], 3, 1)


@pytest.mark.parametrize("bulk,W,H", [(1, 120, 80), (2, 180, 110)])
@pytest.mark.parametrize("unit,eps", [(1.0, 2.0 ** -11), (1.0, 0.01), (2.0 ** -15, 2.0 ** -11), (1e15, 0.5),
                                      (1e-30, 0.01), (1e33, 0.01)])
def test_viewer_next_to_the_nearest(F, orc, bulk, W, H, unit, eps):  # noqa: F811
    L = 7
    d, o, pofa = both(F, orc, near_and_far(bulk), L)
    assert fits(F, pofa, d)
    z = (np.floor(np.float32(0.02) * 2.0 ** (L + 8)) + 0.5 - eps) / 2.0 ** (L + 8)
    compare(F, orc, d, o, pofa, [depth_view(0.0, L, W, H, unit, (0.5, 0.5, z))], (0.0, 1.0 / 256))


def faint_scene(copies):
    """Objects of low opacity (pixels end late), several times in place."""
    mesh = S.cube_scene(6000, 21, scale_range=(0.05, 0.3), ground=8)
    rgba = (mesh.rgba & np.uint32(0x00FFFFFF)) | np.uint32(5 << 24)
    return S.Mesh(np.concatenate([mesh.pos] * copies), np.concatenate([rgba] * copies),
                  np.concatenate([mesh.tri + k * mesh.n_vert for k in range(copies)]).astype(np.uint32),
                  np.concatenate([mesh.obj] * copies))


# depth 5: 12 copies are more fragments than its workspace has boxes for
WAYS = [(7, 1, True), (5, 12, False)]


@pytest.mark.parametrize("L,copies,tiles", WAYS)
@pytest.mark.parametrize("unit", [1.0, 2.0 ** -15, 1e15])
def test_viewer_inside_the_scene(F, orc, unit, L, copies, tiles):  # noqa: F811
    d, o, pofa = both(F, orc, faint_scene(copies), L)
    assert fits(F, pofa, d) == tiles
    views = [depth_view(t, L, 70, 40, unit, at) for t in (0.0, 33.0) for at in ((0.5, 0.5, 0.5), (0.4, 0.4, 0.27))]
    compare(F, orc, d, o, pofa, views, (0.0, 1.0 / 256))


@pytest.mark.parametrize("L,copies,tiles", WAYS)
@pytest.mark.parametrize("unit", [3e34, 6e34])
def test_depths_that_overflow(F, orc, unit, L, copies, tiles):  # noqa: F811
    """Finite and infinite depths in one view, and with the larger unit pixels
    whose nearest depth is infinite: those fragments are met in array order."""
    d, o, pofa = both(F, orc, faint_scene(copies), L)
    assert fits(F, pofa, d) == tiles
    g = 2.0 ** (L + 8)
    views = [depth_view(t, L, 70, 40, unit * 8192 / g, (0.5, 0.5, -0.4)) for t in (0.0, 33.0)]
    assert all(np.isfinite(v.m).all() for v in views)
    compare(F, orc, d, o, pofa, views, (0.0, 1.0 / 256))


@pytest.mark.parametrize("L,copies,tiles", WAYS)
@pytest.mark.parametrize("far,unit", [(1e6, 2.0 ** -15), (1e5, 2.0 ** -15), (1e7, 1.0)])
def test_distant_viewer(F, orc, far, unit, L, copies, tiles):  # noqa: F811
    """Depths rounded to a few values across the whole scene: ties by array
    index between octants on top of each other."""
    d, o, pofa = both(F, orc, faint_scene(copies), L)
    assert fits(F, pofa, d) == tiles
    views = [depth_view(t, L, 70, 40, unit, (0.5, 0.5, -0.4)) for t in (0.0, 33.0)]
    for v in views:
        v.m[2, 3] += np.float32(far)
    compare(F, orc, d, o, pofa, views, (0.0, 1.0 / 256))
