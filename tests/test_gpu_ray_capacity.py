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
