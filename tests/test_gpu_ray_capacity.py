"""Ray casting arrays of no capacity: nothing is met, and every pixel of the
caller's image is written all the same."""
from __future__ import annotations

import pytest

from paper_2211_15460_amd import scenes as S
from tests.gpu_util import run_capture, run_compact
from tests.test_gpu_ray_tiles import F  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,frags", [(0, 0), (0, 1 << 16), (64, 0)])
@pytest.mark.parametrize("L", [1, 5])
@pytest.mark.parametrize("mode", [0, 1])
def test_arrays_without_capacity(F, L, rows, frags, mode):  # noqa: F811
    """No table rows (the scene's, or a table the caller left out), no
    records, or neither: the image comes out zero over what it held."""
    import torch
    mesh = S.cube_scene(200, 31, scale_range=(0.1, 0.3), ground=4)
    d = F.desc(F.FHV_POFL, levels=L)
    *_, lists = run_capture(F, mesh, d, frags)
    _, pofa = run_compact(F, lists, d, rows)
    assert (pofa.cap_occ, pofa.cap_frag) == (rows, frags)
    views = [S.cube_view(t, L, 45, 31, splat_px=1) for t in (0.0, 40.0)]
    out = torch.full((2, 31, 45, 4), 7.5, dtype=torch.float32, device="cuda")
    F.raycast(pofa, d, views, mode=mode, out=out)
    torch.cuda.synchronize()
    assert int(torch.count_nonzero(out).item()) == 0


@pytest.mark.parametrize("L", [4, 7])
@pytest.mark.parametrize("mode", [0, 1])
def test_tiles_leave_the_walks_memory(F, L, mode):  # noqa: F811
    """A capacity too large for the workspace's boxes, fragments that fit: the
    octree walk is prepared for but does nothing, and the workspace past the
    boxes (16 bytes each, after 256) stays as it was."""
    import torch
    mesh = S.cube_scene(40, 32, scale_range=(0.1, 0.3), ground=4)
    d = F.desc(F.FHV_POFL, levels=L)
    need = F.raycast_workspace(d)
    *_, lists = run_capture(F, mesh, d, need * 4)   # 64 fragments a box
    n = int(lists.counter.item())
    _, pofa = run_compact(F, lists, d)
    boxes, nodes, top = 0, -(-n // 64), 0
    while True:   # chunks, groups of 64, ... down to 512 at level 1 or above
        boxes += nodes
        if top >= 1 and nodes <= 512:
            break
        nodes, top = -(-nodes // 64), top + 1
    assert 0 < 256 + 16 * boxes < need
    ws = torch.full((need,), 0xA5, dtype=torch.uint8, device="cuda")
    out = F.raycast(pofa, d, [S.cube_view(20.0, L, 64, 48, splat_px=1)], mode=mode, ws=ws)
    torch.cuda.synchronize()
    assert int(torch.count_nonzero(out).item()) > 0
    assert bool((ws[256 + 16 * boxes:] == 0xA5).all().item())
