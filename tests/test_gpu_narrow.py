"""GPU: frontier steps taken by one block and by many (the searches of gamma,
the opening loop and the assignment, and the MIS sweeps).  A step moves from
one to the other at 2,048 vertices and at 16,384 arcs; stars cross each limit
by one vertex, ER graphs start with a frontier on either side of it, and
both alternate within one solve.  Every output must equal the oracle's."""
import pytest
import torch

import graphgen as gg

from gpu_util import assert_solve_equal

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"


@pytest.mark.parametrize("wmax", [None, 5])
@pytest.mark.parametrize("n", [1024, 1025, 2048, 2049, 2050, 16384, 16385, 16386])
def test_star_around_the_limits(n, wmax):
    """The hub's row has n - 1 arcs; from the hub the next frontier has n - 1
    vertices (unit weights)."""
    print(f"[narrow] star {n} wmax {wmax}", flush=True)
    g = gg.with_problem(gg.star(n, wmax, n), n, cost="uniform", cost_hi=30)
    assert_solve_equal(g, 8, 3)


@pytest.mark.parametrize("n,deg,wmax", [(2047, 7, 10), (2048, 8, None), (2049, 8, 10), (4096, 4, None),
                                        (4099, 9, 100), (6000, 3, 255)])
def test_er_around_the_limits(n, deg, wmax):
    """Every vertex a facility: gamma starts from n seeds."""
    print(f"[narrow] er {n} deg {deg} wmax {wmax}", flush=True)
    g = gg.with_problem(gg.er(n, deg, n, wmax=wmax), n, cost="uniform", cost_hi=200)
    assert_solve_equal(g, 8, 5)


@pytest.mark.parametrize("luby", [False, True])
@pytest.mark.parametrize("directed", [False, True])
def test_hubs_and_long_rows(directed, luby):
    """A power law with rows above the wide steps' queueing limits, few
    expensive facilities, so that the sweeps cover most of the graph."""
    import paper_1503_03635_amd as fl
    g = gg.with_problem(gg.rmat(13, 16 << 13, 9, wmax=20, directed=directed), 9, cost="lognormal", fac_frac=0.1)
    assert_solve_equal(g, 8, 7, flags=(fl.FL_FLAG_LUBY_MIS if luby else 0) |
                       (fl.FL_FLAG_DIRECTED if directed else 0))
