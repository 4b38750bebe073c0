"""The splat against the oracle, bit for bit, at the octree depths where its
packed positions and its walk change form: depth 1 and 7 (a position's z
starts in the low word), 8 (it no longer does), 10 with more than 512 groups of
chunks (the walk starts above the groups); footprints of one and more pixels,
ragged views, parts off screen and behind the viewer, matrices that are not
finite."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2211_15460_amd import scenes as S
from tests.gpu_util import run_capture, run_compact, run_splat
from tests.test_gpu_splat_tiles import F  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("levels", [1, 7, 8, 10])
def test_splat_at_depth(F, orc, levels):  # noqa: F811
    mesh = S.cube_scene(20000, 31)
    d = F.desc(F.FHV_POFL, levels=levels)
    cap = 1 << 23
    _, _, _, cnt, lists = run_capture(F, mesh, d, cap)
    assert cnt <= cap and (levels < 10 or cnt > 512 * 4096)
    g, pofa = run_compact(F, lists, d)
    print(f"splat depth {levels}: {cnt} fragments", flush=True)
    views = [S.cube_view(20.0 + 30.0 * i, levels, 250, 131, splat_px=k) for i, k in enumerate((1, 2, 17))]
    for r, c, v in ((2, 3, -1.5), (0, 3, 140.0), (1, 1, np.nan), (0, 0, np.inf), (1, 3, -3e9)):
        w = S.cube_view(35.0, levels, 250, 131, splat_px=1 if r else 3)
        m = w.m.copy()
        m[r, c] = m[r, c] + np.float32(v)
        views.append(S.View(m, 250, 131, w.splat_px))
    gr, gd, gc = run_splat(F, pofa, d, views)
    orr, od, oc = orc.splat(1, g["key"], g["frag"], views, levels=levels)
    assert np.array_equal(gc, oc) and np.array_equal(gr, orr)
    assert np.array_equal(gd.view(np.uint32), od.view(np.uint32))
    assert oc[:3].any()
