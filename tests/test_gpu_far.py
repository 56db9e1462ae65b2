"""GPU: graphs whose farthest pair is (n - 1) edges of the largest weight apart.
The last level marks its neighbours once more, up to a weight beyond that."""
import numpy as np
import pytest
import torch

import graphgen as gg

from gpu_util import assert_sketch_equal, assert_solve_equal

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"


@pytest.mark.parametrize("w", [1, 17, 18, 24, 100, 255])
@pytest.mark.parametrize("n", [2, 3, 4, 9, 70])
def test_equal_weights_on_a_path(n, w):
    print(f"[far] path {n} weight {w}", flush=True)
    g = gg.path(n, 2)
    g.w = np.full_like(g.w, w)
    gg.with_problem(g, n, cost="uniform", cost_hi=40)
    assert_sketch_equal(g, 8, 3)
    assert_solve_equal(g, 8, 3)
