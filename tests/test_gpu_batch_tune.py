"""What the batch autotuner may choose: launch choices that reach a launch."""
from __future__ import annotations

import pytest

from tests.test_gpu_batch import F, run_batch, scene_views, small_batch  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def test_tuner_leaves_the_splat_alone(F):  # noqa: F811
    """splat_wg reaches no launch; timings of equal launches must not choose
    it (a graph is kept per choice of the others)."""
    try:
        F.set_tuning(8, 16, 5)
        run_batch(F, small_batch(9, [3000, 800]), scene_views(2, 2, 1), flags=F.FHV_BATCH_TUNE)
        t = F.get_tuning()
        assert t["splat_wg"] == 5
        assert t["tile_w"] in (8, 16, 32) and t["raster_wg"] in (4, 8, 16, 32)
    finally:
        F.set_tuning()
