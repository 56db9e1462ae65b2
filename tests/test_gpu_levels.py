"""GPU: sketch levels of every size class.  In a star the hub's level at
distance 1 has as many candidates as there are leaves, and every leaf's at
distance 2 one fewer: a level decided by comparing pairs (up to 12 for two
tasks per wave), by one sort, in chunks of 64, by octave buckets and past a
buffer of survivors.  In a complete bipartite graph every candidate of a level
arrives once per vertex of the other side.  Sketches must equal the oracle's
bit for bit."""
import numpy as np
import pytest
import torch

import graphgen as gg

from gpu_util import assert_sketch_equal

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    assert torch.cuda.is_available(), "GPU tests need an MI355X"


def _flags(dense):
    import paper_1503_03635_amd as fl
    return 0 if dense else fl.FL_FLAG_NO_DENSE


@pytest.mark.parametrize("dense", [True, False])
@pytest.mark.parametrize("k", [8, 32, 33, 64, 128])
def test_star_levels(k, dense):
    for leaves in (11, 12, 13, 14, 31, 32, 33, 34, 63, 64, 65, 66, 127, 129, 513, 1025, 1200, 2049, 9000):
        print(f"[levels] star {leaves} k {k} dense {dense}", flush=True)
        assert_sketch_equal(gg.star(leaves + 1, None, leaves), k, leaves, flags=_flags(dense))


@pytest.mark.parametrize("dense", [True, False])
@pytest.mark.parametrize("k", [16, 64, 128])
def test_copies_of_every_candidate(k, dense):
    for a, b, wmax in ((13, 40, None), (33, 70, None), (65, 300, None), (200, 150, None), (40, 90, 2), (300, 20, 3)):
        print(f"[levels] bipartite {a} {b} w {wmax} k {k} dense {dense}", flush=True)
        u = np.repeat(np.arange(a), b)
        v = a + np.tile(np.arange(b), a)
        g = gg.from_edges(a + b, u, v, wmax, np.random.Generator(np.random.PCG64(a)), name="bipartite")
        assert_sketch_equal(g, k, a, flags=_flags(dense))


@pytest.mark.parametrize("k", [16, 64, 128])
@pytest.mark.parametrize("make", [
    lambda: gg.er(2000, 8, 2, wmax=10), lambda: gg.rmat(11, 16 << 11, 9), lambda: gg.star(3001, 7, 1),
    lambda: gg.grid(40, 41, wmax=4), lambda: gg.rmat(11, 16 << 11, 4, wmax=100, directed=True)],
    ids=["er w10", "rmat unit", "star w7", "grid w4", "rmat directed w100"])
def test_marks_by_vertex(make, k, monkeypatch):
    """Graphs whose arc positions exceed 32 bits mark vertices; the hook takes
    small ones there."""
    import paper_1503_03635_amd as fl
    g = make()
    directed = fl.FL_FLAG_DIRECTED if getattr(g, "directed", False) else 0
    monkeypatch.setenv("FL_TEST_MARK_VERTICES", "1")
    print(f"[levels] marks by vertex n {g.n} k {k}", flush=True)
    got = assert_sketch_equal(g, k, 7, flags=fl.FL_FLAG_NO_DENSE | directed)
    monkeypatch.delenv("FL_TEST_MARK_VERTICES")
    want = assert_sketch_equal(g, k, 7, flags=fl.FL_FLAG_NO_DENSE | directed)
    for key in got:
        assert np.array_equal(got[key], want[key]), key
