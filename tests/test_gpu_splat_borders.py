"""Splats and rays whose tiles' borders lie on the faces of the fragments' boxes:
the octree's planes at pixel borders, per axis and view direction, boxes in units
of one and of several grid steps, and per-pixel arrays seen from the front.
Against the oracle."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2211_15460_amd import scenes as S
from tests.test_gpu_bricks import F  # noqa: F401  (fixture)
from tests.test_gpu_ray_tiles import both, compare
from tests.test_gpu_splat_loads import against_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [3, 8, 9])
@pytest.mark.parametrize("theta", [0.0, 90.0, 180.0, 45.0])
def test_borders_on_octree_planes(F, orc, L, theta):  # noqa: F811
    """64 pixels over the cube, so that every octree plane down to depth 6 is a
    pixel border, and many are a tile's or a sub-tile's (a dense sheet makes
    the tiles split)."""
    g = np.random.default_rng(L)
    mesh = S.cube_scene(400, 60 + L, scale_range=(0.02, 0.1) if L > 8 else (0.1, 0.4), ground=0 if L > 8 else 8)
    pos = np.floor(mesh.pos * 64) / 64 if L < 9 else mesh.pos
    pos = np.where(g.random(pos.shape) < 0.5, pos, mesh.pos).astype(np.float32)
    mesh = S.Mesh(pos, mesh.rgba, mesh.tri, mesh.obj)
    for side, extent, px in ((128, 1.0, 1), (256, 2.0, 2)):
        views = [S.cube_view(theta, L, side, side, vertical_extent=extent, splat_px=px)]
        assert against_oracle(F, orc, mesh, L, views) > 0
    d, o, pofa = both(F, orc, mesh, L)
    compare(F, orc, d, o, pofa, [S.cube_view(theta, L, 64, 64, vertical_extent=1.0, splat_px=1)], (1.0 / 256,))


def test_pixel_borders(F, orc):  # noqa: F811
    """Per-pixel arrays seen from the front: every position is a pixel centre,
    boxes end half a pixel before the tiles' borders."""
    mesh = S.clip_soup(300, 7)
    for k in (1, 2):
        views = [S.ppfl_view(0.0, 160, 130, splat_px=k), S.ppfl_view(180.0, 160, 130, splat_px=k)]
        assert against_oracle(F, orc, mesh, 0, views, 0, 160, 130) > 0
