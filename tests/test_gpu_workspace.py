"""GPU: the workspace a call reports (fl_stats.workspace_bytes)."""
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
