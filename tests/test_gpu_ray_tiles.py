"""Ray casting by screen tiles (arrays whose boxes fit the workspace) against
the oracle, bit for bit: tiles with more hits than one slab holds, pixels met
hundreds of times, hits of one depth, partly covered tiles and odd sizes, walks
of one and several levels; a scene far from the view and views that see
nothing; and the way chosen by the fragment count where only that fits."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2211_15460_amd import scenes as S
from tests.gpu_util import run_capture, run_compact
from tests.test_gpu_raycast import cast, stacked_planes, with_alpha

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2211_15460_amd import fhv
    fhv.lib()
    return fhv


def both(F, orc, mesh, L, spare=64, cap_occ=None):
    """The oracle's arrays and the GPU's, in a pool of `spare` slots beyond
    the scene's fragments."""
    oh, op, oc = orc.capture_pofl(mesh, L, 6 << 20)
    o = orc.compact(oh, op, oc)
    d = F.desc(F.FHV_POFL, levels=L)
    *_, lists = run_capture(F, mesh, d, int(oc) + spare)
    g, pofa = run_compact(F, lists, d, cap_occ)
    if cap_occ is None:
        assert np.array_equal(g["frag"], o["frag"])
    return d, o, pofa


def fits(F, pofa, d):
    """Whether boxes for the arrays' capacity fit the workspace (16 bytes per
    64 fragments and for the levels above)."""
    chunks = (pofa.cap_frag + 63) // 64
    return 16 * (chunks + chunks // 60 + 4) + 512 < F.raycast_workspace(d)


def compare(F, orc, d, o, pofa, views, taus=(0.0, 1.0 / 256)):
    got = cast(F, pofa, d, views, F.FHV_RAY_NEAREST)
    assert np.array_equal(got, orc.raycast(o["key"], o["frag"], views, d.levels, mode=0)[0])
    for tau in taus:
        want, deepest = orc.raycast(o["key"], o["frag"], views, d.levels, mode=1, tau=tau)
        print(f"tau {tau} deepest pixel {deepest}", flush=True)
        assert np.array_equal(cast(F, pofa, d, views, F.FHV_RAY_BLEND, tau), want)


@pytest.mark.parametrize("W,H", [(1, 1), (16, 16), (17, 15), (160, 96), (333, 50)])
def test_sizes(F, orc, W, H):
    mesh = with_alpha(S.cube_scene(6000, 21, scale_range=(0.05, 0.3), ground=8), 3)
    d, o, pofa = both(F, orc, mesh, 7)
    assert fits(F, pofa, d)
    compare(F, orc, d, o, pofa, [S.cube_view(t, 7, W, H, splat_px=1) for t in (0.0, 33.0, 90.0)])


@pytest.mark.parametrize("planes,alpha", [(40, 12), (40, 0), (9, 3), (30, 255)])
def test_many_hits_per_tile(F, orc, planes, alpha):
    """Squares facing the view, 64 samples of each per pixel: one depth per
    plane, hundreds to thousands of hits per pixel, hundreds of thousands
    per tile."""
    mesh = stacked_planes(planes, alpha, 3)
    d, o, pofa = both(F, orc, mesh, 7)
    assert fits(F, pofa, d)
    compare(F, orc, d, o, pofa, [S.cube_view(t, 7, 70, 40, splat_px=1) for t in (0.0, 15.0)], (0.0, 0.5))


def test_distant_scene(F, orc):
    """The whole scene in a few pixels, at one depth in float: the slabs end
    up divided by array index."""
    mesh = with_alpha(S.cube_scene(20000, 22, scale_range=(0.02, 0.2)), 4)
    d, o, pofa = both(F, orc, mesh, 8)
    assert fits(F, pofa, d)
    views = []
    for scale, depth in ((0.02, 1.0), (0.004, 0.0)):
        v = S.cube_view(30.0, 8, 96, 64, splat_px=1)
        m = v.m.astype(np.float64)
        m[:2] *= scale
        m[0, 3] += 40.3
        m[1, 3] += 30.7
        m[2] *= depth
        m[2, 3] += 1.5
        views.append(S.View(m.astype(np.float32), 96, 64, 1))
    compare(F, orc, d, o, pofa, views)


def test_views_that_see_nothing(F, orc):
    mesh = with_alpha(S.cube_scene(3000, 23, scale_range=(0.05, 0.3), ground=0), 5)
    d, o, pofa = both(F, orc, mesh, 7)
    views = []
    for row, by in ((0, 1e6), (1, -1e6), (2, -1e9)):
        v = S.cube_view(10.0, 7, 40, 24, splat_px=1)
        v.m[row, 3] += np.float32(by)
        views.append(v)
    compare(F, orc, d, o, pofa, views)


@pytest.mark.parametrize("L,n_tri", [(3, 40), (6, 4000)])
def test_way_chosen_by_the_fragment_count(F, orc, L, n_tri):
    """A pool far larger than the workspace has boxes for: the fragments'
    boxes fit (the tiles) or not (the octree walk)."""
    mesh = with_alpha(S.cube_scene(n_tri, 24, scale_range=(0.1, 0.4), ground=4), 6)
    for copies in (1, 12):
        m = S.Mesh(np.concatenate([mesh.pos] * copies), np.concatenate([mesh.rgba] * copies),
                   np.concatenate([mesh.tri + k * mesh.n_vert for k in range(copies)]).astype(np.uint32),
                   np.concatenate([mesh.obj] * copies))
        d, o, pofa = both(F, orc, m, L, spare=1 << 20)
        assert not fits(F, pofa, d)
        compare(F, orc, d, o, pofa, [S.cube_view(t, L, 90, 60, splat_px=1) for t in (0.0, 50.0)], (1.0 / 256,))


def test_truncated_table(F, orc):
    """Fragments of rows that the table does not hold are not met."""
    mesh = with_alpha(S.cube_scene(6000, 25, scale_range=(0.05, 0.3), ground=8), 7)
    d, o, pofa = both(F, orc, mesh, 7, cap_occ=1500)
    end = int(o["off"][1500])
    views = [S.cube_view(t, 7, 120, 70, splat_px=1) for t in (0.0, 60.0)]
    for mode in (0, 1):
        want = orc.raycast(o["key"], o["frag"][:end], views, 7, mode=mode, tau=0.01)[0]
        assert np.array_equal(cast(F, pofa, d, views, mode, 0.01), want)
