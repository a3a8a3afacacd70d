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


# ---------------------------------------------------- connected components

@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, 511, 513, 30011])
@pytest.mark.parametrize("sym", [True, False])
def test_components_of_ragged_sizes(gpu, n, sym):
    """Sparse random graphs around the block and sample sizes: isolated
    vertices, many small components and one large one."""
    for k, m in enumerate((n // 2, n, 3 * n)):
        rng = np.random.default_rng(10 * n + k)
        g = graphgen.from_edges(n, rng.integers(0, n, m), rng.integers(0, n, m), symmetrize=sym)
        assert np.array_equal(gpu.cc(load(gpu, g)).cpu().numpy(), oracle.cc(g.offsets, g.cols)), (n, m, sym)


@pytest.mark.parametrize("sym", [True, False])
@pytest.mark.parametrize("deg", [4, 5, 12, 13, 76, 511, 512, 5000])
def test_components_joined_past_the_sampled_edges(gpu, deg, sym):
    """Stars of equal size joined only through the last edge of each centre's
    row, so that no sampled edge and no large component hides it: rows just
    inside and past the sampled four, the one-lane rows, the wave's and the
    blocks'."""
    k = 6
    src, dst = [], []
    for i in range(k):
        c = i * (deg + 1)
        src += [c] * deg
        dst += list(range(c + 1, c + deg + 1))
    # the centres' largest neighbour: a leaf of the next star, in pairs
    for i in range(0, k, 2):
        src.append(i * (deg + 1))
        dst.append((i + 2) * (deg + 1) - 1)
    n = k * (deg + 1) + 3
    for flip in (False, True):
        a, b = (dst, src) if flip else (src, dst)
        g = graphgen.from_edges(n, np.array(a), np.array(b), symmetrize=sym)
        ref = oracle.cc(g.offsets, g.cols)
        assert len(np.unique(ref)) == k // 2 + 3
        assert np.array_equal(gpu.cc(load(gpu, g)).cpu().numpy(), ref), (deg, sym, flip)


def test_components_of_long_paths(gpu):
    """Paths whose parent links form one long chain: vertices in id order, so
    that every vertex starts under its predecessor, alone and next to a star."""
    n = 60000
    for extra in (0, 4000):
        src = np.r_[np.arange(n - 1), np.full(extra, n)]
        dst = np.r_[np.arange(1, n), n + 1 + np.arange(extra)]
        g = graphgen.from_edges(n + 1 + extra, src, dst, symmetrize=True)
        lab = gpu.cc(load(gpu, g)).cpu().numpy()
        assert np.array_equal(lab, oracle.cc(g.offsets, g.cols)), extra
