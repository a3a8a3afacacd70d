"""Kernels at the sizes where their work split changes: tile and chunk edges,
remainders, the smallest and largest rows of a branch, against the oracle."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

INF = oracle.INF


def load(tg, g, weights=None, tuning=None):
    G = tg.graph_load_csr(g.n, g.offsets, g.cols, weights, symmetric=g.symmetric)
    return tg.partition_by_degree(G, tuning=tuning)


# ------------------------------------------------------------- BFS parents

@pytest.mark.parametrize("place", [0, 3, 4, 67, 68, 131, 132, 499])
def test_parent_at_each_place_of_a_row(gpu, place):
    """The only possible parent at a given place of a 500-long in-row: the
    four lanes of the first look, the two halves of a wave's step, later
    steps and the row's end; unreached in-neighbours around it."""
    d = 500
    u = np.arange(1, d + 1)
    x = d + 1
    g = graphgen.from_edges(d + 2, np.r_[0, u], np.r_[1 + place, np.full(d, x)], symmetrize=False)
    P = load(gpu, g)
    lev, par = gpu.bfs(P, [0, 1 + place], want_parents=True)
    lev, par = lev.cpu().numpy(), par.cpu().numpy()
    for i, r in enumerate((0, 1 + place)):
        assert np.array_equal(lev[i], oracle.bfs(g.offsets, g.cols, r))
        assert np.all((par[i] == -1) == (lev[i] == INF))
        assert par[i][r] == r and par[i][x] == 1 + place
    assert par[0][1 + place] == 0


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 1000])
def test_parents_of_ragged_vertex_counts(gpu, n):
    """Every vertex of a random tree has its tree parent (the only one)."""
    rng = np.random.default_rng(n)
    up = np.array([rng.integers(0, max(v, 1)) for v in range(1, n)], dtype=np.int64)
    g = graphgen.from_edges(n, up, np.arange(1, n), symmetrize=True)
    lev, par = gpu.bfs(load(gpu, g), [0], want_parents=True)
    assert np.array_equal(lev.cpu().numpy()[0], oracle.bfs(g.offsets, g.cols, 0))
    assert np.array_equal(par.cpu().numpy()[0], np.r_[0, up])
