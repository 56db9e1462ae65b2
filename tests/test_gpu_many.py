"""GPU: batches of thousands of tiny graphs, each equal to its solve alone: the
workspace counts what every graph of a union needs, and a MIS step has as many
graphs as one block gathers (2,048) or more."""
import pytest
import torch

import graphgen as gg
import paper_1503_03635_amd as fl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"


def _bases():
    gs = [gg.path(4), gg.grid(2, 3, wmax=4), gg.star(5, 3, 1), gg.er(12, 3, 2, wmax=5), gg.er(20, 4, 3)]
    return [fl.to_device(gg.with_problem(g, i, cost="uniform", cost_hi=20)) for i, g in enumerate(gs)]


def _check(bases, k, count):
    dgs = [bases[i % len(bases)] for i in range(count)]
    seeds = [1 + i // len(bases) for i in range(count)]
    keys = {"open": torch.uint8, "assign": torch.int32, "dist": torch.int32, "open_rung": torch.int32,
            "freeze_rung": torch.int32, "q": torch.float64}
    ends = torch.tensor([d.n for d in dgs]).cumsum(0).tolist()
    whole = {key: torch.zeros(ends[-1], dtype=t, device="cuda") for key, t in keys.items()}
    outs = [{key: t[e - d.n:e] for key, t in whole.items()} for d, e in zip(dgs, ends)]
    got = fl.solve_batch(dgs, k, seeds, 0.1, outputs=outs)
    assert all(r["status"] == 0 for r in got)
    step = max(1, count // 200)
    for i in list(range(0, count, step)) + [count - 1]:
        want = fl.solve(dgs[i], k, seeds[i], 0.1, diagnostics=True)
        for key in keys:
            assert torch.equal(got[i][key], want[key]), (i, key)
        for key in ("total_cost", "n_open", "n_unreachable"):
            assert got[i][key] == want[key], (i, key)
        for key in ("rungs", "mis_rounds", "gamma"):
            assert got[i]["stats"][key] == want["stats"][key], (i, key)


@pytest.mark.parametrize("count", [40, 6000, 24000])
def test_many_tiny_graphs(count):
    """Three workers share a batch, a third of the graphs each."""
    print(f"[many] {count} graphs", flush=True)
    _check(_bases(), 4, count)


@pytest.mark.parametrize("each", [1, 2, 3, 255, 2047, 2048, 2049, 5001])
def test_ranges_of_a_step(each):
    """Cycles of four vertices and one cost, sketches exact: all facilities of
    all graphs open in one rung, a single step of `each` ranges per worker."""
    print(f"[many] {each} ranges", flush=True)
    ring = fl.to_device(gg.with_problem(gg.grid(2, 2), 1, cost="uniform", cost_lo=5, cost_hi=5))
    assert (fl.solve(ring, 4, 1, diagnostics=True)["open_rung"].unique().numel()) == 1
    _check([ring], 4, 3 * each)
