"""The training step's layer checks with the weight and bias gradients held to the
rounding bound of the order in which one launch for all layers sums them: the
steps of a wave one after the other, eight waves pairwise, a tile's workgroups
in four interleaved groups."""
from __future__ import annotations

import pytest

from oracle import unet as U
from tests import test_gpu_fill_trace as T
from tests.test_gpu_fill_trace import F  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

WAVES, GROUPS, MIN_STEPS = 8, 768, 8


def plan(levels, N, H, W):
    """{(grid pixels, cin, cout): (steps per wave, workgroups per tile, up)}: the
    steps of all layers' tiles cut into runs of one length, a step of a
    transposed convolution counting twice."""
    layers = []
    for kind, lvl, ci, co in grids(levels):
        h, w = H >> lvl, W >> lvl
        cin = (ci + 7) // 8 * 8
        strips = (w + 7) // 8
        assert h * w * max(cin, 8 * co) < 1 << 27   # beyond, rows are padded to groups of strips
        steps = (N * strips + 3) // 4 * h
        layers.append((N * h * w, cin, co, kind == "t2", (co // 32) * ((cin + 31) // 32), steps))
    cost = lambda up: 2 if up else 1
    total = sum(tiles * steps * cost(up) for *_, up, tiles, steps in layers)
    parts = lambda up, steps, per: -(-steps * cost(up) // (per * WAVES))
    per = max(MIN_STEPS, total // (GROUPS * WAVES))
    while sum(t * parts(up, s, per) for *_, up, t, s in layers) > GROUPS and per < total:
        per += per // 32 + 1
    out = {}
    for P, ci, co, up, _, steps in layers:
        p = parts(up, steps, per)
        out[P, ci, co] = (-(-steps // (p * WAVES)), p, up)
    return out


def grids(levels):
    """(kind, level of the step grid, cin, cout) of every layer but the head."""
    specs = U.layer_specs(levels)
    lvl = [l for l in range(levels) for _ in range(2)]
    for l in reversed(range(levels - 1)):
        lvl += [l + 1, l, l]
    assert len(specs) == len(lvl) + 1
    return [(s[0], l, s[1], s[2]) for s, l in zip(specs, lvl)]


@pytest.mark.parametrize("levels,N,H,W", [(1, 1, 8, 16), (2, 1, 18, 130), (3, 2, 20, 132),
                                          pytest.param(4, 8, 256, 256, marks=pytest.mark.slow)])
def test_gradients_within_their_own_order(F, monkeypatch, levels, N, H, W):  # noqa: F811
    p = plan(levels, N, H, W)

    def wgrad(P, ci, co):   # two products of 16 pixels and the sum before, per step
        per, parts, _ = p[P, ci, co]
        return 34 * per + 3 + (parts + 3) // 4 + 2

    def bgrad(P):   # pairs, then one after the other: 8 a step, 32 in a transposed one; two lanes
        per = max(8 * a + 1 if not up else 32 * a + 1 for (q, _, _), (a, _, up) in p.items() if q in (P, P // 4))
        parts = max(b for (q, _, _), (_, b, _) in p.items() if q in (P, P // 4))
        return per + 1 + 3 + (parts + 3) // 4 + 2

    monkeypatch.setattr(T, "wgrad_depth", wgrad)
    monkeypatch.setattr(T, "bgrad_depth", bgrad)
    T.test_every_layer_of_a_training_step(F, levels, N, H, W)
