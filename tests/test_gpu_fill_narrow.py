"""Training steps at sizes where the weight gradients' pixel strips go wrong
first: levels narrower than a strip of 8 pixels (a group of strips then spans
several images), widths just past a strip and past a group of four, single
rows and single pixels, one level only. Every tensor of every layer against
fp64 on the tensors it read, as in the layer tests; the summation bound holds
for any order (as many roundings as there are terms)."""
import pytest

from tests import test_gpu_fill_trace as T
from tests.test_gpu_fill_trace import F  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("levels,N,H,W", [(1, 5, 3, 1), (1, 2, 33, 9), (2, 7, 2, 6), (3, 5, 12, 20), (4, 3, 8, 8),
                                          (3, 1, 4, 260), (2, 1, 130, 34), (4, 1, 72, 200)])
def test_layers_of_narrow_training_steps(F, monkeypatch, levels, N, H, W):  # noqa: F811
    monkeypatch.setattr(T, "wgrad_depth", lambda P, ci, co: P + 2)
    monkeypatch.setattr(T, "bgrad_depth", lambda P: P + 2)
    T.test_every_layer_of_a_training_step(F, levels, N, H, W)
