"""GPU: the workspace a call reports (fl_stats.workspace_bytes), and with it
which rows the MIS sweeps of a weighted graph read: a copy in weight-class order
(8 bytes per arc and direction) where the call's own reservation has room, the
rows as they are elsewhere, whatever was solved before."""
import numpy as np
import pytest
import torch

import graphgen as gg
import paper_1503_03635_amd as fl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"


def _bytes(g, solve=None, **kw):
    return (solve or fl.solve)(fl.to_device(g), 8, 1, **kw)["stats"]["workspace_bytes"]


@pytest.mark.parametrize("wmax", [100, 255])
def test_workspace_holds_the_selection(wmax):
    """The MIS sweeps hold a pending label and a list entry per vertex and
    distance slot (max weight + 1 of them)."""
    g = gg.with_problem(gg.er(20000, 6, 1, wmax=wmax), 1, cost="uniform", cost_hi=200)
    assert g.w.max() == wmax
    print(f"[workspace] wmax {wmax}", flush=True)
    for solve in (fl.solve, fl.solve_static):
        assert _bytes(g, solve) >= 8 * g.n * (wmax + 1)


def _circulant(n, off, wmax, directed):
    """Arcs to the vertices at the offsets `off` (closed under negation where
    undirected)."""
    src = torch.arange(n, device="cuda")[:, None]
    dst = ((src + torch.tensor(off).cuda()) % n).sort(dim=1).values
    w = 1 + (src * dst + src + dst) % wmax  # the same in both directions
    cost = np.random.default_rng(3).integers(1, 400, n).astype(np.int32)
    return fl.DeviceGraph(n=n, row_ptr=torch.arange(n + 1, device="cuda") * len(off),
                          col=dst.to(torch.int32).reshape(-1), w=w.to(torch.int32).reshape(-1),
                          fac_cost=torch.from_numpy(cost).cuda(), directed=directed)


def test_rows_do_not_depend_on_earlier_calls():
    """38 million arcs out of 60,000 vertices, weights 1..4: the reservation has
    no room for the copies of both directions."""
    dg = _circulant(60000, range(1, 641), 4, True)
    large = fl.to_device(gg.with_problem(gg.er(300000, 6, 1, wmax=255), 1, cost="uniform", cost_hi=200))
    fl.release_workspace()
    before = fl.solve(dg, 4, 1)
    fl.solve(large, 8, 1)
    after = fl.solve(dg, 4, 1)
    assert before["stats"]["workspace_bytes"] == after["stats"]["workspace_bytes"]
    assert before["total_cost"] == after["total_cost"]


def test_fixed_workspace_without_the_copy():
    """30 million arcs: a call's own workspace holds the ordered rows, the
    library's fixed one does not."""
    dg = _circulant(29600, [*range(-500, 0), *range(1, 501)], 16, False)
    own, fixed = (solve(dg, 4, 1) for solve in (fl.solve, fl.solve_static))
    assert own["stats"]["workspace_bytes"] - fixed["stats"]["workspace_bytes"] >= 8 * dg.n_arcs
    for key in ("open", "assign", "dist"):
        assert torch.equal(own[key], fixed[key]), key
