"""GPU: searches of many wide iterations (frontiers beyond one block, on grids
whose distances take hundreds of them), and frontiers of every remainder of a
block's four waves."""
import numpy as np
import pytest
import torch

import graphgen as gg

from gpu_util import assert_solve_equal

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"


@pytest.mark.parametrize("wmax,few", [(9, 0.01), (None, 0.002), (4, 1.0)])
def test_long_searches(wmax, few):
    """Costs far above the edge weights: few facilities open, and their
    distances spread over the grid iteration by iteration."""
    print(f"[searches] grid 250x300 wmax {wmax}", flush=True)
    g = gg.with_problem(gg.grid(250, 300, wmax=wmax, seed=1), 1, cost="uniform", cost_lo=20000, cost_hi=60000,
                        fac_frac=few)
    got, _ = assert_solve_equal(g, 8, 3)
    assert 0 < got["n_open"] < 200


@pytest.mark.parametrize("leaves", [2049, 2051, 2112, 4095, 8193, 8255])
def test_remainders_of_a_block(leaves):
    """A hub's leaves are the next frontier and have one more arc each, to a
    vertex of their own: every wave of the wide step appends what its few
    vertices lead to."""
    n = 2 * leaves + 1
    ids = np.arange(1, leaves + 1)
    g = gg.from_edges(n, np.r_[np.zeros(leaves, np.int64), ids], np.r_[ids, ids + leaves], 7,
                      np.random.Generator(np.random.PCG64(leaves)), name="broom")
    g = gg.with_problem(g, leaves, cost="uniform", cost_lo=300, cost_hi=900, fac_frac=0.01)
    print(f"[searches] broom {leaves}", flush=True)
    assert_solve_equal(g, 8, 5)
