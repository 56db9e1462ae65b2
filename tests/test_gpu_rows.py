"""GPU: the passes over rows.  Validation and the reverse arcs take equal ranges
of arcs, whatever rows they cross.  MIS sweeps read rows in weight-class order:
rows up to 4,096 arcs are ordered by a wave, longer ones by a block; a
workspace without room for the ordered rows leaves them as they are.
Whole-number outputs, so all must be equal."""
import numpy as np
import pytest
import torch

import graphgen as gg

from gpu_util import assert_solve_equal

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"


@pytest.mark.parametrize("wmax", [2, 16, 255])
@pytest.mark.parametrize("n", [65, 66, 4096, 4097, 4098, 5122, 70001])
def test_hub_row_lengths(n, wmax):
    """The hub's row has n - 1 arcs: one group of 64 and one more, the longest
    row of a wave and one more, a block's last part with two arcs."""
    print(f"[rows] star {n} wmax {wmax}", flush=True)
    g = gg.with_problem(gg.star(n, wmax, n), n, cost="uniform", cost_hi=400)
    assert_solve_equal(g, 8, 3)


@pytest.mark.parametrize("directed", [False, True])
@pytest.mark.parametrize("wmax", [1, 3, 255])
def test_directions_and_weights(wmax, directed):
    import paper_1503_03635_amd as fl
    print(f"[rows] rmat wmax {wmax} directed {directed}", flush=True)
    g = gg.with_problem(gg.rmat(12, 12 << 12, 5, wmax=wmax, directed=directed), 5, cost="lognormal", fac_frac=0.2)
    assert_solve_equal(g, 8, 11, flags=fl.FL_FLAG_DIRECTED if directed else 0)


def test_no_room_for_the_copy():
    """29.6 million arcs: the library's own 256 MiB workspace holds the sketch
    rounds but has no room for the ordered rows (8 bytes per arc); a call's
    own workspace has."""
    import paper_1503_03635_amd as fl
    n, half = 29600, 500
    off = torch.cat([torch.arange(-half, 0), torch.arange(1, half + 1)]).cuda()
    src = torch.arange(n, device="cuda")[:, None]
    dst = ((src + off) % n).sort(dim=1).values
    w = 1 + (src * dst + src + dst) % 16  # the same in both directions
    cost = np.random.default_rng(3).integers(1, 400, n).astype(np.int32)
    dg = fl.DeviceGraph(n=n, row_ptr=torch.arange(n + 1, device="cuda") * (2 * half),
                        col=dst.to(torch.int32).reshape(-1), w=w.to(torch.int32).reshape(-1),
                        fac_cost=torch.from_numpy(cost).cuda())
    a = fl.solve(dg, 4, 1, diagnostics=True)
    b = fl.solve_static(dg, 4, 1, diagnostics=True)
    for key in ("open", "assign", "dist", "open_rung", "freeze_rung", "q"):
        assert torch.equal(a[key], b[key]), key
    for key in ("mis_rounds", "rungs", "gamma"):
        assert a["stats"][key] == b["stats"][key], key
    assert a["n_open"] == b["n_open"] and a["total_cost"] == b["total_cost"]


def _spread(n, gap, extra):
    """A star on every gap-th vertex, so that whole groups of 64 rows are empty,
    and a path over the first `extra` vertices."""
    at = np.arange(0, n, gap)
    a = np.concatenate([np.zeros(len(at) - 1, np.int64), np.arange(extra - 1)])
    b = np.concatenate([at[1:], np.arange(1, extra)])
    return gg.from_edges(n, a, b, 7, np.random.Generator(np.random.PCG64(n)), name="spread")


@pytest.mark.parametrize("n,gap,extra", [(9000, 63, 2), (9000, 64, 65), (9000, 65, 130), (70000, 1000, 3)])
def test_empty_rows_between(n, gap, extra):
    print(f"[rows] spread {n} {gap} {extra}", flush=True)
    g = gg.with_problem(_spread(n, gap, extra), n, cost="uniform", cost_hi=30)
    assert_solve_equal(g, 8, 3)


@pytest.mark.parametrize("what", ["weight", "head", "loop"])
@pytest.mark.parametrize("at", ["first", "group", "next", "last"])
def test_one_wrong_arc_is_refused(at, what):
    import paper_1503_03635_amd as fl
    g = gg.with_problem(gg.er(3000, 9, 2, wmax=10), 2, cost="uniform", cost_hi=30)
    dg = fl.to_device(g)
    assert fl.solve(dg, 8, 1)["status"] == 0
    m = dg.n_arcs
    i = {"first": 0, "group": m // 128 * 64 - 1, "next": m // 128 * 64, "last": m - 1}[at]
    if what == "weight":
        dg.w[i] = 11
    elif what == "head":
        dg.col[i] = dg.n
    else:
        dg.col[i] = int(np.searchsorted(np.asarray(g.row_ptr, np.int64), i, side="right") - 1)
    out = fl.solve(dg, 8, 1, check=False)
    assert out["rc"] == fl._lib.FL_EINVAL
