"""GPU: the opening loop's device control and the MIS lists past the sizes one
block takes: more rungs than the ladder window holds, more facilities opened in
a rung than a block seeds, more facilities, clients and touched vertices of a
rung than a block lists; alone and as part of a union."""
import pytest
import torch

import graphgen as gg

from gpu_util import assert_solve_equal

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"


@pytest.mark.parametrize("eps", [0.004, 0.002])
def test_more_rungs_than_the_ladder_window(eps):
    g = gg.with_problem(gg.er(120, 4, 3, wmax=10), 3, cost="uniform", cost_hi=300)
    got, _ = assert_solve_equal(g, 8, 3, eps=eps)
    assert got["stats"]["rungs"] > 2048


def _equal_costs(n, deg, wmax):
    return gg.with_problem(gg.er(n, deg, n, wmax=wmax), n, cost="uniform", cost_lo=3, cost_hi=3)


@pytest.mark.parametrize("n,deg,wmax", [(2049, 4, None), (17000, 3, None), (17000, 3, 4), (70000, 3, None),
                                        (70000, 3, 3)])
def test_large_rungs(n, deg, wmax):
    """Equal costs: most facilities open and most clients freeze in few rungs."""
    print(f"[rungs] er {n} {deg} wmax {wmax}", flush=True)
    assert_solve_equal(_equal_costs(n, deg, wmax), 8, 5)


def test_large_rungs_in_a_union():
    import paper_1503_03635_amd as fl
    gs = [_equal_costs(70000, 3, 3), gg.with_problem(gg.er(300, 5, 1, wmax=10), 1, cost="uniform", cost_hi=200),
          _equal_costs(17000, 3, None)]
    dgs = [fl.to_device(g) for g in gs]
    alone = [fl.solve(d, 8, 5, diagnostics=True) for d in dgs]
    union = fl.solve_batch(dgs, 8, 5, diagnostics=True)
    for a, b in zip(alone, union):
        for key in ("open", "assign", "dist", "open_rung", "freeze_rung", "q"):
            assert torch.equal(a[key], b[key]), key
        assert a["total_cost"] == b["total_cost"] and a["stats"]["mis_rounds"] == b["stats"]["mis_rounds"]
