"""GPU: facilities that are not clients.  Until a client is in finite reach of
an open facility every rung of the opening loop begins with the stall check;
here rungs behind such a check open more facilities than one block seeds (2,048)
and their searches take more wide iterations than one chain launches; alone and
as part of a union."""
import numpy as np
import pytest
import torch

import graphgen as gg
import paper_1503_03635_amd as fl

from gpu_util import assert_solve_equal

pytestmark = pytest.mark.gpu
BLOCK_SEEDS = 2048


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"


def _sites(g, sites, costs):
    """Facilities at `sites`, every other vertex a client."""
    g.fac_cost = np.full(g.n, gg.NOT_FACILITY, np.uint32)
    g.fac_cost[sites] = costs
    g.is_client = np.ones(g.n, np.uint8)
    g.is_client[sites] = 0
    return g


def _existing_sites(wmax=None):
    """2,700 sites open at cost 0, in the first rung, on a grid of 90,000
    vertices, and 60 costly ones."""
    g = gg.grid(300, 300, wmax=wmax, seed=4)
    at = np.random.default_rng(1).choice(g.n, 2760, replace=False)
    return _sites(g, at, np.r_[np.zeros(2700, np.uint32), np.full(60, 400, np.uint32)])


def _equal_sites(n, deg, wmax):
    """Half of the vertices are facilities of one small cost, all weights are
    multiples of 50: most open in the rung that first reaches a neighbour."""
    g = gg.er(n, deg, n, wmax=wmax)
    g.w = g.w * 50
    return _sites(g, np.arange(0, n, 2), 4)


def _largest_rung(open_rung):
    t, count = np.unique(open_rung[open_rung < fl.FL_RUNG_END], return_counts=True)
    return int(t[count.argmax()]), int(count.max())


@pytest.mark.parametrize("wmax", [None, 3])
def test_existing_sites(wmax):
    print(f"[sites] grid 300x300 wmax {wmax}", flush=True)
    got, _ = assert_solve_equal(_existing_sites(wmax), 8, 3)
    t, count = _largest_rung(got["open_rung"])
    assert t == 1 and count > BLOCK_SEEDS


@pytest.mark.parametrize("n,deg,wmax", [(17000, 3, 1), (17000, 3, 4), (70000, 4, 3)])
def test_equal_sites(n, deg, wmax):
    print(f"[sites] er {n} {deg} wmax {wmax}", flush=True)
    got, _ = assert_solve_equal(_equal_sites(n, deg, wmax), 8, 5)
    t, count = _largest_rung(got["open_rung"])
    assert t > 8 and count > BLOCK_SEEDS


@pytest.mark.parametrize("eps", [0.1, 0.01])
def test_checks_fall_due_late(eps):
    """Two components: in one every vertex is a client and a cheap facility and
    freezes early, in the other the facilities are no clients and dear, so that
    the check first falls due many rungs into the loop."""
    a, b = gg.er(400, 5, 1, wmax=4), gg.grid(25, 40, wmax=9, seed=2)
    g = gg.disjoint_union(a, b)
    at = a.n + np.arange(0, b.n, 7)
    _sites(g, at, np.random.default_rng(3).integers(500, 4000, len(at)))
    g.fac_cost[:a.n] = 3
    print(f"[sites] late, eps {eps}", flush=True)
    got, _ = assert_solve_equal(g, 8, 2, eps=eps)
    assert got["freeze_rung"][:a.n].max() + 20 < got["open_rung"][at][got["open_rung"][at] < fl.FL_RUNG_END].min()


def test_sites_in_a_union():
    gs = [_existing_sites(3), gg.with_problem(gg.er(300, 5, 1, wmax=10), 1, cost="uniform", cost_hi=200),
          _equal_sites(17000, 3, 4), _existing_sites(),
          gg.with_problem(gg.er(9000, 4, 2, wmax=4), 2, cost="uniform", cost_lo=5, cost_hi=5)]
    dgs = [fl.to_device(g) for g in gs]
    alone = [fl.solve(d, 8, 5, diagnostics=True) for d in dgs]
    union = fl.solve_batch(dgs, 8, 5, diagnostics=True)
    for a, b in zip(alone, union):
        for key in ("open", "assign", "dist", "open_rung", "freeze_rung", "q"):
            assert torch.equal(a[key], b[key]), key
        assert a["total_cost"] == b["total_cost"] and a["stats"]["mis_rounds"] == b["stats"]["mis_rounds"]
