"""Splats whose tiles queue chunk counts around a draw step (four chunks a wave,
sixteen waves), so that the loads ahead of the draws end inside a step. Against
the oracle."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2211_15460_amd import scenes as S
from tests.gpu_util import run_capture, run_compact, run_splat
from tests.test_gpu_bricks import F  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def against_oracle(F, orc, mesh, L, views, mode=1, W=0, H=0):  # noqa: F811
    if mode:
        d, o = F.desc(F.FHV_POFL, levels=L), orc.compact(*orc.capture_pofl(mesh, L, 4 << 20))
    else:
        d, o = F.desc(F.FHV_PPFL, W, H), orc.compact(*orc.capture_ppfl(mesh, W, H, 4 << 20))
    n = o["frag"].shape[0]
    *_, lists = run_capture(F, mesh, d, n + 5)
    _, pofa = run_compact(F, lists, d)
    want = orc.splat(mode, o["key"], o["frag"], views, levels=L) if mode else \
        orc.splat(0, o["key"], o["frag"], views, width_cap=W)
    for got, w in zip(run_splat(F, pofa, d, views), want):
        assert np.array_equal(got, w)
    return n


@pytest.mark.parametrize("n_tri", [1, 40, 300, 1200, 5000])
@pytest.mark.parametrize("px", [1, 3])
def test_chunks_per_tile(F, orc, n_tri, px):  # noqa: F811
    g = np.random.default_rng(n_tri)
    c = g.random((n_tri, 1, 3))
    pos = np.clip(c + g.normal(0, 0.05, (n_tri, 3, 3)), 0, 0.9999).reshape(-1, 3).astype(np.float32)
    mesh = S.Mesh(pos, g.integers(0, 2 ** 32, 3 * n_tri, dtype=np.uint32),
                  np.arange(3 * n_tri, dtype=np.uint32).reshape(-1, 3), None)
    views = [S.cube_view(t, 6, 70, 64, splat_px=px) for t in (0.0, 77.0)]
    assert against_oracle(F, orc, mesh, 6, views) > 0
