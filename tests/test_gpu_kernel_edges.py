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


# ------------------------------------------------- multi-source supersteps

def core_and_tail(scale, tail, hub=0, seed=3):
    """An R-MAT core (large frontiers: pulled) with a path hung on its largest
    vertex (small frontiers for `tail` more levels) and `hub` leaves on the
    path's end (one row past the block sizes, far from the core)."""
    core = graphgen.rmat(scale, seed=seed)
    deg = np.diff(core.offsets)
    src = np.repeat(np.arange(core.n), deg)
    c = graphgen.max_degree_vertex(core)
    path = np.r_[c, core.n + np.arange(tail)]
    end = path[-1]
    leaves = core.n + tail + np.arange(hub)
    n = core.n + tail + hub
    a = np.r_[src, path[:-1], np.full(hub, end)]
    b = np.r_[core.cols, path[1:], leaves]
    return graphgen.from_edges(n, a, b, symmetrize=True), c, int(end)


@pytest.mark.parametrize("tail,hub", [(3, 0), (40, 700), (252, 0), (253, 0), (254, 3), (300, 9000)])
def test_batched_levels_and_distances_past_one_byte(gpu, tail, hub):
    """Pulled, mixed and pushed supersteps in one run, frontiers that grow
    again after shrinking, and levels on both sides of the one-byte limit;
    a second run on the same engine starts from its kept buffers."""
    g, c, end = core_and_tail(9, tail, hub)
    w = graphgen.weights(g, seed=4)
    for tuning in (None, {"bfs_do": 0}, {"hub_min_deg": 64, "block_min_deg": 32, "wave_min_deg": 16,
                                         "g16_min_deg": 6, "g4_min_deg": 2, "hub_chunk": 256}):
        P = load(gpu, g, w, tuning)
        for k, count in enumerate((64, 5, 1)):
            roots = ([end, c] + graphgen.sample_roots(g, 62, seed=k).tolist())[:count]
            lev = gpu.bfs_batched(P, roots).cpu().numpy()
            dist = gpu.sssp_batched(P, roots).cpu().numpy()
            for i in sorted({0, 1, count // 2, count - 1} & set(range(count))):
                assert np.array_equal(lev[i], oracle.bfs(g.offsets, g.cols, roots[i])), (tuning, count, i)
                assert np.array_equal(dist[i], oracle.sssp(g.offsets, g.cols, w, roots[i])), (tuning, count, i)


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1023, 1025])
@pytest.mark.parametrize("sym", [True, False])
def test_batched_on_ragged_vertex_counts(gpu, n, sym):
    rng = np.random.default_rng(n)
    m = 5 * n
    g = graphgen.from_edges(n, rng.integers(0, n, m), rng.integers(0, n, m), symmetrize=sym)
    w = graphgen.weights(g, seed=5)
    P = load(gpu, g, w)
    roots = rng.integers(0, n, 64).tolist()
    lev, dist = gpu.bfs_batched(P, roots).cpu().numpy(), gpu.sssp_batched(P, roots).cpu().numpy()
    for i in range(0, 64, 7):
        assert np.array_equal(lev[i], oracle.bfs(g.offsets, g.cols, roots[i]))
        assert np.array_equal(dist[i], oracle.sssp(g.offsets, g.cols, w, roots[i]))


@pytest.mark.parametrize("leaves", [3, 600])
def test_pulled_distances_that_do_not_fit(gpu, leaves):
    """Overflowing candidates in the pulled supersteps of a symmetric graph,
    from rows of both splits: the verdict names the root whose distances do
    not fit, and a candidate that overflows beside one that fits is no error."""
    big = 2**31 - 10
    # a clique carries the frontier; vertex 9 hangs on leaf rows by edges too
    # heavy for anything but a direct start
    a, b = np.triu_indices(8, 1)
    src = np.r_[a, np.full(leaves, 8), 0, 8]
    dst = np.r_[b, 9 + np.arange(leaves), 8, 9 + leaves]
    g = graphgen.from_edges(10 + leaves, src, dst, symmetrize=True)
    row = np.repeat(np.arange(g.n), np.diff(g.offsets))
    heavy = (row == 9 + leaves) | (g.cols == 9 + leaves)
    w = np.where(heavy, big, 1000).astype(np.int32)
    P = load(gpu, g, w)
    far = 9 + leaves
    with pytest.raises(gpu.TGError) as ei:
        gpu.sssp_batched(P, [8, 3])
    assert ei.value.code == gpu.TG_ERANGE and "root 3" in str(ei.value)
    ok = gpu.sssp_batched(P, [8]).cpu().numpy()[0]
    assert ok[far] == big and ok[0] == 1000
    # a lighter way round: the overflowing candidate no longer matters
    g2 = graphgen.from_edges(g.n, np.r_[src, 3], np.r_[dst, far], symmetrize=True)
    row2 = np.repeat(np.arange(g2.n), np.diff(g2.offsets))
    pair = ((row2 == far) & (g2.cols == 8)) | ((row2 == 8) & (g2.cols == far))
    w2 = np.where(pair, big, 1000).astype(np.int32)
    got = gpu.sssp_batched(load(gpu, g2, w2), [8, 3, far]).cpu().numpy()
    for i, r in enumerate((8, 3, far)):
        assert np.array_equal(got[i], oracle.sssp(g2.offsets, g2.cols, w2, r))


@pytest.mark.parametrize("deg", [3, 15, 17, 100, 511, 512, 1500])
@pytest.mark.parametrize("sym,roots", [(True, 5), (True, 6), (True, 64), (False, 16), (False, 17), (False, 64)])
def test_distances_of_many_slots_that_do_not_fit(gpu, deg, sym, roots):
    """Overflowing candidates with more slots in flight than are walked edge by
    edge: pulled rows of each split and pushed ones, edges that many slots
    share and edges with one; `far` hangs on `deg` vertices of a random core by
    edges that only a search from one of them can take."""
    big = 2**31 - 10
    rng = np.random.default_rng(deg)
    core = deg + 200
    far, one, two = core, core + 1, core + 2  # and a path far from the core, for one slot
    a, b = rng.integers(0, core, 10 * core), rng.integers(0, core, 10 * core)
    ring = np.arange(core)
    near = np.arange(deg)  # the vertices next to `far`
    src = np.r_[a, ring, near, one, two]
    dst = np.r_[b, (ring + 1) % core, np.full(deg, far), two, core + 3]
    g = graphgen.from_edges(core + 4, src, dst, symmetrize=sym)
    row = np.repeat(np.arange(g.n), np.diff(g.offsets))
    w = np.where((row < core) & (g.cols < core), 1000, big).astype(np.int32)
    P = load(gpu, g, w)
    inside = rng.integers(0, deg, roots - 2).tolist()

    def same(P, w, rs):
        got = gpu.sssp_batched(P, rs).cpu().numpy()
        pulls = gpu.tg_last_stats()["pull_supersteps"]
        # (the search on the short path ends early: five leave four)
        assert pulls > 0 if sym and roots > 5 else sym or pulls == 0
        for i in sorted({0, 1, len(rs) // 2, len(rs) - 2, len(rs) - 1}):
            assert np.array_equal(got[i], oracle.sssp(g.offsets, g.cols, w, rs[i])), i

    good = inside + [two, near[0]]
    same(P, w, good)  # `two` is the middle of its path
    for bad, name in ((deg + 50, deg + 50), (one, one)):
        with pytest.raises(gpu.TGError) as ei:
            gpu.sssp_batched(P, inside[:3] + [bad] + inside[3:] + [two])
        assert ei.value.code == gpu.TG_ERANGE and f"root {name}" in str(ei.value)
    with pytest.raises(gpu.TGError) as ei:
        gpu.sssp_batched(P, (deg + np.arange(roots)).tolist())
    assert ei.value.code == gpu.TG_ERANGE
    # one of the edges is light: candidates overflow, then the vertex is reached
    light = ((row == 0) & (g.cols == far)) | ((row == far) & (g.cols == 0))
    w2 = np.where(light, 1000, w).astype(np.int32)
    same(load(gpu, g, w2), w2, (deg + np.arange(roots)).tolist())
    same(P, w, good)  # nothing of the failed calls is left


@pytest.mark.parametrize("deg", [1, 63, 64, 65, 511, 513, 2049])
def test_batched_betweenness_rows_of_each_split(gpu, deg):
    """Two hubs sharing `deg` middle vertices (every row sum a multiple of the
    tile, or one off), a tail behind each, and isolated vertices."""
    mid = 2 + np.arange(deg)
    t = deg + 2
    src = np.r_[np.zeros(deg, int), np.ones(deg, int), 0, t, 1, t + 2]
    dst = np.r_[mid, mid, t, t + 1, t + 2, t + 3]
    n = t + 6
    for sym in (True, False):
        g = graphgen.from_edges(n, src, dst, symmetrize=sym)
        srcs = [0, 1, 2, t + 1, t + 3, deg + 1, n - 1] + list(range(2, min(2 + deg, 70)))
        ref = oracle.bc(g.offsets, g.cols, srcs)
        for tuning in (None, {"hub_min_deg": 50, "block_min_deg": 20, "wave_min_deg": 8, "g16_min_deg": 4,
                              "g4_min_deg": 2, "hub_chunk": 256}):
            got = gpu.bc_batched(load(gpu, g, None, tuning), srcs).cpu().numpy().astype(np.float64)
            assert np.all(np.abs(got - ref) <= 1e-5 * np.abs(ref) + 1e-6 * max(ref.max(), 1.0)), (sym, tuning)


def test_batched_betweenness_deep_graph_grows_its_queue(gpu):
    """A path: every source reaches each vertex at its own level, far more
    queue entries than vertices."""
    n = 700
    g = graphgen.from_edges(n, np.arange(n - 1), np.arange(1, n), symmetrize=True)
    srcs = list(range(0, n, 11))
    ref = oracle.bc(g.offsets, g.cols, srcs)
    P = load(gpu, g)
    for _ in range(2):
        got = gpu.bc_batched(P, srcs).cpu().numpy().astype(np.float64)
        assert np.all(np.abs(got - ref) <= 1e-5 * np.abs(ref) + 1e-6 * ref.max())


def test_batched_distances_past_2_to_26_vertices(gpu):
    """64 slots a vertex are more than 2^32 entries: a slot's distances are
    cleared when it retires, so that the next search in it starts afresh."""
    import torch
    n, k = (1 << 26) + 5, 1000
    i = np.arange(k)
    col = np.stack([i - 1, i + 1], 1).ravel()
    deg = np.zeros(n + 1, dtype=np.int64)
    deg[1:k + 1] = 2
    deg[1] = deg[k] = 1
    G = gpu.graph_load_csr(n, np.cumsum(deg), col[(col >= 0) & (col < k)], np.full(2 * k - 2, 300),
                           symmetric=True, validate=False)
    P = gpu.partition_by_degree(G)
    out = torch.empty((2, n), dtype=torch.int32, device="cuda")
    for r in (0, k - 1, 500):
        gpu.sssp_batched(P, [r, n - 1], out)
        assert np.array_equal(out[0, :k].cpu().numpy(), 300 * np.abs(i - r)), r
        assert int((out[0] != INF).sum()) == k and int((out[1] != INF).sum()) == 1


# ------------------------------------- calls routed to the 64-slot engines

@pytest.mark.parametrize("sym", [True, False])
@pytest.mark.parametrize("count", [0, 1, 2, 3, 4, 8, 63, 64, 65, 130])
def test_engine_and_single_searches_agree(gpu, sym, count):
    """bfs, sssp and bc with the engines chosen by rule, forced and refused:
    repeated and isolated roots, chunks of 64 and their remainders."""
    g = graphgen.rmat(11, symmetrize=sym, seed=6)
    w = graphgen.weights(g, seed=7)
    iso = int(np.argmin(np.diff(g.offsets)))
    roots = (graphgen.sample_roots(g, 60, seed=9).tolist() + [iso, iso, 5, 5] + list(range(100)))[:count]
    ref_l = ref_d = None
    for tuning in ({"bfs_batch_roots": 0, "sssp_batch_roots": 0}, None, {"bfs_batch_roots": 1, "sssp_batch_roots": 1},
                   {"bfs_lanes": 2, "sssp_lanes": 2}):
        P = load(gpu, g, w, tuning)
        if count == 0:
            # an empty output has no address: refused on either route
            for call in (gpu.bfs, gpu.sssp):
                with pytest.raises(gpu.TGError) as ei:
                    call(P, roots)
                assert ei.value.code == gpu.TG_EINVAL
            continue
        lev, dist = gpu.bfs(P, roots).cpu().numpy(), gpu.sssp(P, roots).cpu().numpy()
        if ref_l is None:
            ref_l, ref_d = lev, dist
            for i in range(0, count, 16):
                assert np.array_equal(lev[i], oracle.bfs(g.offsets, g.cols, roots[i]))
                assert np.array_equal(dist[i], oracle.sssp(g.offsets, g.cols, w, roots[i]))
        assert np.array_equal(lev, ref_l) and np.array_equal(dist, ref_d), tuning
    got = gpu.bc(P, roots).cpu().numpy().astype(np.float64)
    ref = oracle.bc(g.offsets, g.cols, roots)
    assert np.all(np.abs(got - ref) <= 1e-5 * np.abs(ref) + 1e-6 * max(np.abs(ref).max(), 1.0))


def test_overflow_verdict_is_the_same_on_both_routes(gpu):
    g = graphgen.from_edges(3, [0, 1], [1, 2], symmetrize=True)
    w = np.full(g.nnz, 2**31 - 10, dtype=np.int32)
    for tuning in ({"sssp_batch_roots": 0}, {"sssp_batch_roots": 1}, None):
        P = load(gpu, g, w, tuning)
        with pytest.raises(gpu.TGError) as ei:
            gpu.sssp(P, [1, 0])
        assert ei.value.code == gpu.TG_ERANGE
        assert gpu.sssp(P, [1]).cpu().numpy().tolist() == [[2**31 - 10, 0, 2**31 - 10]]


# -------------------------------------------- statistics of every route

def stats_of(tg, call):
    call()
    return tg.tg_last_stats()


@pytest.mark.parametrize("sym", [True, False])
@pytest.mark.parametrize("count", [1, 3, 40, 70])
def test_bfs_statistics_on_every_route(gpu, sym, count):
    """Top-down throughout, the edges scanned are the out-edges of what each
    search reached; with bottom-up steps every vertex that joined in one was
    expanded in neither or one of them.  One workgroup per root, the 64-slot
    engine and single searches."""
    g = graphgen.rmat(10, symmetrize=sym, seed=4)
    deg = np.diff(g.offsets)
    roots = graphgen.sample_roots(g, count, seed=5).tolist()
    reached = [oracle.bfs(g.offsets, g.cols, r) != INF for r in roots]
    verts, edges = sum(int((m & (deg > 0)).sum()) for m in reached), sum(int(deg[m].sum()) for m in reached)
    keys = {"roots", "supersteps", "edges_scanned", "vertices_expanded", "bottom_up_edges_checked", "bottom_up_steps",
            "bottom_up_vertices_examined", "lanes"}
    for route in ({"bfs_batch_roots": 1}, {"bfs_batch_roots": 0}):
        P = load(gpu, g, None, {**route, "bfs_do": 0})
        for call in (gpu.bfs, gpu.bfs_batched):
            st = stats_of(gpu, lambda: call(P, roots))
            assert keys <= set(st), route
            assert (st["edges_scanned"], st["vertices_expanded"]) == (edges, verts), (route, call)
            assert st["bottom_up_steps"] == st["bottom_up_edges_checked"] == st["bottom_up_vertices_examined"] == 0
    # (workgroups: a frontier past the queue is looked for all the same)
    for tuning in ({"bfs_do": 0, "bfs_batch_roots": -1}, {"bfs_batch_roots": -1, "bfs_do": 1}, {"bfs_batch_roots": 1},
                   {"bfs_batch_roots": 0}):
        st = stats_of(gpu, lambda: gpu.bfs(load(gpu, g, None, tuning), roots))
        assert keys <= set(st) and st["roots"] == count and st["lanes"] >= min(count, 2), tuning
        # (none where every superstep of the engine is pulled)
        assert 0 <= st["edges_scanned"] <= edges and 0 <= st["vertices_expanded"] <= verts, tuning
        if st["bottom_up_steps"] == 0:
            assert (st["edges_scanned"], st["vertices_expanded"]) == (edges, verts), tuning
        else:
            assert st["edges_scanned"] < edges, tuning
            assert 0 < st["bottom_up_vertices_examined"] <= g.n * st["bottom_up_steps"], tuning
            assert st["bottom_up_vertices_examined"] <= st["bottom_up_edges_checked"] + g.n * st["bottom_up_steps"]
            assert st["bottom_up_edges_checked"] <= g.nnz * st["bottom_up_steps"], tuning
    assert stats_of(gpu, lambda: gpu.bfs(load(gpu, g), roots))["bottom_up_steps"] > 0


def test_pulled_edges_are_counted(gpu):
    """A star's leaves each look at their one in-neighbour, the hub, when it
    is on the frontier, and the far hub's row is read to its end."""
    leaves = 3000
    g = graphgen.from_edges(leaves + 1, np.zeros(leaves, int), np.arange(1, leaves + 1), symmetrize=True)
    for tuning in (None, {"bfs_batch_roots": 1}):
        P = load(gpu, g, None, tuning)
        # every leaf is unvisited but the root of the search; then none is
        st = stats_of(gpu, lambda: gpu.bfs(P, [0, 0]))
        assert st["supersteps"] in (2, 4)
        if tuning is None:
            assert st["bottom_up_edges_checked"] == st["bottom_up_vertices_examined"] == 2 * leaves
        else:  # shared: a leaf looks once for both
            assert st["bottom_up_edges_checked"] == st["bottom_up_vertices_examined"] == leaves


@pytest.mark.parametrize("sym", [True, False])
@pytest.mark.parametrize("count", [1, 4, 5, 20, 64, 70])
def test_sssp_statistics_on_every_route(gpu, sym, count):
    """Every reached vertex relaxes its out-edges at least once for each
    search; on a path from its end exactly once."""
    g = graphgen.rmat(10, symmetrize=sym, seed=4)
    w = graphgen.weights(g, seed=1)
    deg = np.diff(g.offsets)
    roots = graphgen.sample_roots(g, count, seed=5).tolist()
    reached = [oracle.bfs(g.offsets, g.cols, r) != INF for r in roots]
    verts, edges = sum(int((m & (deg > 0)).sum()) for m in reached), sum(int(deg[m].sum()) for m in reached)
    n = 300
    path = graphgen.from_edges(n, np.arange(n - 1), np.arange(1, n), symmetrize=sym)
    keys = {"roots", "supersteps", "relaxations", "activations", "pull_supersteps", "heavy_pull_edges_checked",
            "heavy_pull_vertices", "lanes"}
    for tuning in (None, {"sssp_batch_roots": 1}, BUCKETS, {"sssp_batch_roots": 0}):
        st = stats_of(gpu, lambda: gpu.sssp(load(gpu, g, w, tuning), roots))
        assert keys <= set(st) and st["roots"] == count and 1 <= st["lanes"] <= count, tuning
        if not st["heavy_pull_edges_checked"]:  # (else a bucket's heavy edges are not relaxed from its members)
            assert st["activations"] >= verts and st["relaxations"] >= edges, tuning
        if tuning == {"sssp_batch_roots": 1}:
            assert (st["pull_supersteps"] > 0) == (sym and count > 4)
        st = stats_of(gpu, lambda: gpu.sssp(load(gpu, path, np.ones(path.nnz, np.int32), tuning), [0] * count))
        if not st["heavy_pull_edges_checked"]:
            has = int((np.diff(path.offsets) > 0).sum())
            assert st["relaxations"] == count * path.nnz, tuning
            # (the single searches count a vertex once per pass, light and heavy)
            assert count * has <= st["activations"] <= count * has * (2 if tuning == {"sssp_batch_roots": 0} else 1)
    st = stats_of(gpu, lambda: gpu.sssp_batched(load(gpu, g, w), roots))
    assert keys <= set(st) and st["relaxations"] >= edges and st["edges_read"] >= edges / min(count, 64)


# ------------------------------------------- one workgroup per BFS root

@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 63, 64, 65, 1023, 1024, 1025, 32768, 65536, 65537])
@pytest.mark.parametrize("sym", [True, False])
def test_workgroup_bfs_of_each_size(gpu, n, sym):
    """Bitmap word pairs, the 1024-vertex sweep, the largest graphs it takes
    and the first it does not; a star and a random graph in one, so that the
    queue overflows and rows of all lengths are looked through."""
    rng = np.random.default_rng(n)
    k = n // 3
    src = np.r_[np.zeros(k, int), rng.integers(0, n, 3 * n)]
    dst = np.r_[np.arange(k), rng.integers(0, max(n // 2, 1), 3 * n)]
    g = graphgen.from_edges(n, src, dst, symmetrize=sym)
    roots = [0, n - 1, n // 2, 0] + rng.integers(0, n, 3).tolist()
    lev, par = gpu.bfs(load(gpu, g), roots, want_parents=True)
    lev, par = lev.cpu().numpy(), par.cpu().numpy()
    only = gpu.bfs(load(gpu, g), roots).cpu().numpy()
    assert np.array_equal(only, lev)
    for i, r in enumerate(roots):
        assert np.array_equal(lev[i], oracle.bfs(g.offsets, g.cols, r)), (i, r)
        v = np.nonzero((lev[i] != INF) & (np.arange(n) != r))[0]
        assert par[i][r] == r and np.all(par[i][lev[i] == INF] == -1)
        assert np.all(lev[i][par[i][v]] == lev[i][v] - 1)


@pytest.mark.parametrize("tail", [1, 252, 253, 254, 255, 400])
def test_workgroup_bfs_past_its_deepest_level(gpu, tail):
    """Levels up to and past what a byte holds (the launched supersteps take
    over), with a frontier beyond the queue at the end of the path."""
    g, c, end = core_and_tail(8, tail, hub=3000)
    for roots in ([c], [end, c, 0], [end] * 65):
        lev, par = gpu.bfs(load(gpu, g), roots, want_parents=True)
        lev = lev.cpu().numpy()
        assert np.array_equal(lev, gpu.bfs(load(gpu, g), roots).cpu().numpy())
        for i in {0, len(roots) - 1}:
            assert np.array_equal(lev[i], oracle.bfs(g.offsets, g.cols, roots[i])), (tail, i)


# ------------------------------------- SSSP for a few roots, in rounds

@pytest.mark.parametrize("n", [1, 2, 16, 17, 64, 65, 1025, 5000])
@pytest.mark.parametrize("sym", [True, False])
@pytest.mark.parametrize("top", [1, 255, 100000])
def test_round_sssp_of_each_size(gpu, n, sym, top):
    """Packed and two-array edges, ragged spans of 1, 4 and 16 vertices, a row
    past the 1024-thread block's turn, several roots per launch."""
    rng = np.random.default_rng(n)
    src = np.r_[np.zeros(n, int), rng.integers(0, n, 4 * n)]
    dst = np.r_[np.arange(n), rng.integers(0, max(n // 2, 1), 4 * n)]
    g = graphgen.from_edges(n, src, dst, symmetrize=sym)
    w = graphgen.weights(g, seed=n, lo=1, hi=top)
    for tuning in (None, {"hub_min_deg": 64, "block_min_deg": 32, "wave_min_deg": 16, "g16_min_deg": 6,
                          "g4_min_deg": 2, "hub_chunk": 256}):
        P = load(gpu, g, w, tuning)
        for roots in ([n - 1], [0, n // 2, 0, n - 1, n // 3]):
            dist = gpu.sssp(P, roots).cpu().numpy()
            for i, r in enumerate(roots):
                assert np.array_equal(dist[i], oracle.sssp(g.offsets, g.cols, w, r)), (tuning, roots, i)


@pytest.mark.parametrize("n", [12, 13, 14, 17, 40, 130, 3000])
def test_round_sssp_chunks_end_anywhere(gpu, n):
    """Paths whose number of rounds is on either side of a chunk's end, and a
    root without edges (no round relaxes anything)."""
    g = graphgen.from_edges(n + 1, np.arange(n - 1), np.arange(1, n), symmetrize=True)
    w = graphgen.weights(g, seed=n)
    P = load(gpu, g, w)
    for _ in range(2):
        dist = gpu.sssp(P, [0, n]).cpu().numpy()
        for i, r in enumerate((0, n)):
            assert np.array_equal(dist[i], oracle.sssp(g.offsets, g.cols, w, r)), r
        assert gpu.sssp(P, [n]).cpu().numpy()[0].tolist() == [INF] * n + [0]


@pytest.mark.parametrize("leaves", [2, 600])
@pytest.mark.parametrize("sym", [True, False])
def test_round_sssp_overflow(gpu, leaves, sym):
    """Overflowing candidates from short rows and from a block's row: an error
    only where the vertex stays unreached."""
    big = 2**31 - 10
    far = leaves + 2
    src = np.r_[0, np.full(leaves, 1), 1]
    dst = np.r_[1, 2 + np.arange(leaves), far]
    g = graphgen.from_edges(far + 1, src, dst, symmetrize=sym)
    row = np.repeat(np.arange(g.n), np.diff(g.offsets))
    w = np.where((row == far) | (g.cols == far), big, 50).astype(np.int32)
    P = load(gpu, g, w)
    with pytest.raises(gpu.TGError) as ei:
        gpu.sssp(P, [0])
    assert ei.value.code == gpu.TG_ERANGE
    assert np.array_equal(gpu.sssp(P, [1]).cpu().numpy()[0], oracle.sssp(g.offsets, g.cols, w, 1))
    g2 = graphgen.from_edges(g.n, np.r_[src, 0], np.r_[dst, far], symmetrize=sym)
    row2 = np.repeat(np.arange(g2.n), np.diff(g2.offsets))
    pair = ((row2 == 1) & (g2.cols == far)) | ((row2 == far) & (g2.cols == 1))
    w2 = np.where(pair, big, 50).astype(np.int32)
    assert np.array_equal(gpu.sssp(load(gpu, g2, w2), [0]).cpu().numpy()[0], oracle.sssp(g2.offsets, g2.cols, w2, 0))


# ------------------------------------------ PageRank over sliced columns

# None: rows walked whole; the others name a schedule, which takes the classes:
# as they are, without a table of hot contributions, with one line of it per
# class, and with one workgroup per class.
PR_TUNINGS = [None, {"pr_xcd": 1}, {"pr_lds_verts": 0}, {"pr_lds_verts": 32}, {"pr_grid": 8}]


def check_pagerank(tg, g, tuning, iters=4):
    """All terms are positive; per iteration a rank carries at most the
    rounding of its contributions and of its partial sums, and one more when it
    is written: (2 iters + 1) 2^-24, and one 2^-24 for the sums in 64 bits."""
    P = load(tg, g, tuning=tuning)
    for dangling in ("uniform", "drop"):
        want = oracle.pagerank(g.offsets, g.cols, iterations=iters, dangling=dangling)
        for _ in range(2):
            r = tg.pagerank(P, iterations=iters, dangling=dangling).cpu().numpy().astype(np.float64)
            assert np.all(np.abs(r - want) <= (2 * iters + 2) * 2.0**-24 * want), (tuning, dangling)


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 255, 257, 511, 512, 513, 1025, 30011])
@pytest.mark.parametrize("sym", [True, False])
def test_pagerank_slices_of_ragged_sizes(gpu, n, sym):
    """Windows, slices and classes that end anywhere; isolated vertices."""
    rng = np.random.default_rng(n)
    for m in (0, n // 2, 9 * n):
        g = graphgen.from_edges(n, rng.integers(0, n, m), rng.integers(0, n, m), symmetrize=sym)
        for tuning in PR_TUNINGS:
            check_pagerank(gpu, g, tuning)


@pytest.mark.parametrize("around", [32, 128, 1024, 2048, 9 * 1024])
@pytest.mark.parametrize("sym", [True, False])
def test_pagerank_rows_around_each_split(gpu, around, sym):
    """Rows just below and above the longest of a slice, one piece and several
    (whole rows, and their eighths in the classes)."""
    rng = np.random.default_rng(around)
    pool = 24000
    if around * 8 <= pool:
        lens = np.r_[around + np.arange(-2, 3), 8 * around + np.arange(-48, 49, 8)]
    else:
        lens = around + np.arange(-64, 65, 16)
    src = np.concatenate([rng.choice(pool, k, replace=False) for k in lens])
    dst = pool + np.repeat(np.arange(lens.size), lens)
    back = rng.integers(0, pool, 40000)
    src, dst = np.r_[src, back], np.r_[dst, rng.integers(0, pool + lens.size, 40000)]
    g = graphgen.from_edges(pool + lens.size, src, dst, symmetrize=sym)
    for tuning in PR_TUNINGS:
        check_pagerank(gpu, g, tuning)


def test_pagerank_rows_of_one_class(gpu):
    """Symmetric, so that ids follow degrees: 128 hubs of equal degree hold
    four classes, rows of only those leave the other classes empty."""
    n, hubs = 6000, 128
    src = np.tile(np.arange(hubs), n - hubs)
    dst = np.repeat(np.arange(hubs, n), hubs)
    keep = (src + dst) % 3 > 0
    g = graphgen.from_edges(n, src[keep], dst[keep], symmetrize=True)
    for tuning in PR_TUNINGS:
        check_pagerank(gpu, g, tuning)


# The classes on graphs that are walked whole unless "pr_whole" says otherwise.
PR_CLASSES = [{"pr_whole": 0}, {"pr_whole": 0, "pr_lds_verts": 0}, {"pr_whole": 0, "pr_lds_verts": 32},
              {"pr_whole": 0, "pr_grid": 8}]


def pagerank_kernels(tg, P):
    tg.tg_set_timing(True)
    try:
        tg.pagerank(P, iterations=2)
        return {k for k in tg.tg_last_stats() if k.endswith("_n")}
    finally:
        tg.tg_set_timing(False)


def test_small_graphs_are_walked_whole_whatever_else_is_tuned(gpu):
    """Naming a key of the classes does not cost a small graph its one launch
    an iteration; "pr_whole" chooses."""
    g = graphgen.rmat(10)
    for tuning in PR_TUNINGS:
        assert pagerank_kernels(gpu, load(gpu, g, tuning=tuning)) == {"pr_gather_n"}, tuning
    assert pagerank_kernels(gpu, load(gpu, g, tuning={"pr_whole": 0})) == {"pr_slice_gather_n", "pr_combine_n"}
    assert pagerank_kernels(gpu, load(gpu, g, tuning={"pr_whole": 1, "pr_grid": 8})) == {"pr_gather_n"}
    with pytest.raises(gpu.TGError):
        load(gpu, g, tuning={"pr_whole": 2})


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 255, 257, 511, 512, 513, 1025, 30011])
@pytest.mark.parametrize("sym", [True, False])
def test_pagerank_classes_of_ragged_sizes(gpu, monkeypatch, n, sym):
    monkeypatch.setitem(globals(), "PR_TUNINGS", PR_CLASSES)
    test_pagerank_slices_of_ragged_sizes(gpu, n, sym)


@pytest.mark.parametrize("around", [32, 128, 1024, 2048, 9 * 1024])
@pytest.mark.parametrize("sym", [True, False])
def test_pagerank_class_rows_around_each_split(gpu, monkeypatch, around, sym):
    monkeypatch.setitem(globals(), "PR_TUNINGS", PR_CLASSES)
    test_pagerank_rows_around_each_split(gpu, around, sym)


def test_pagerank_classes_left_empty(gpu, monkeypatch):
    monkeypatch.setitem(globals(), "PR_TUNINGS", PR_CLASSES)
    test_pagerank_rows_of_one_class(gpu)


@pytest.mark.parametrize("lds", [0, 100, 40960])
def test_pagerank_class_variants(gpu, lds):
    """R-MAT hubs past a piece in every class, and runs that agree to the bit."""
    for g in (graphgen.rmat(14), graphgen.rmat(12, symmetrize=False)):
        check_pagerank(gpu, g, {"pr_whole": 0, "pr_lds_verts": lds, "pr_grid": 64}, iters=10)
        P = load(gpu, g, tuning={"pr_whole": 0, "pr_lds_verts": lds, "pr_grid": 64})
        a, b = (gpu.pagerank(P, iterations=10).cpu().numpy() for _ in range(2))
        assert np.array_equal(a, b)


# -------------------------- SSSP by buckets for several roots at once

BUCKETS = {"sssp_batch_roots": 1 << 20}  # never the engine: the bucket schedule


@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 1025, 16383, 16384, 16385, 32768])
@pytest.mark.parametrize("sym", [True, False])
def test_bucket_sssp_of_ragged_sizes(gpu, n, sym):
    """Words and collecting blocks (16384 vertices) that end anywhere, bins
    that begin and end inside a block, full and partial groups of roots."""
    rng = np.random.default_rng(n)
    m = 5 * n
    g = graphgen.from_edges(n, np.r_[np.zeros(n, int), rng.integers(0, n, m)],
                            np.r_[np.arange(n), rng.integers(0, max(n // 2, 1), m)], symmetrize=sym)
    w = graphgen.weights(g, seed=n)
    bins = {"hub_min_deg": 64, "block_min_deg": 32, "wave_min_deg": 16, "g16_min_deg": 6, "g4_min_deg": 2}
    want = {r: oracle.sssp(g.offsets, g.cols, w, r) for r in (0, n // 3, n // 2, n - 1)}
    for tuning in (BUCKETS, {**BUCKETS, **bins}, {**BUCKETS, "sssp_delta": 255, "sssp_hpull": 0},
                   {**BUCKETS, "sssp_delta": 24, "sssp_hpull": 100000}):
        P = load(gpu, g, w, tuning)
        for roots in ([n - 1], [0, n // 2, 0, n - 1, n // 3, 0, 0, n // 2], [n // 3, 0, n - 1] * 6):
            dist = gpu.sssp(P, roots).cpu().numpy()
            for i, r in enumerate(roots):
                assert np.array_equal(dist[i], want[r]), (tuning, roots, i)


@pytest.mark.parametrize("leaves", [2047, 2048, 2049, 4096, 4097, 40000])
@pytest.mark.parametrize("top", [1, 8, 255])
def test_bucket_sssp_hub_chunks(gpu, leaves, top):
    """Two hubs whose rows end around a chunk's end, all light, some light,
    and few light edges; leaves joined in a ring give longer ways round."""
    a, b = 0, 1
    leaf = 2 + np.arange(leaves)
    src = np.r_[np.full(leaves, a), np.full(leaves - 1, b), leaf]
    dst = np.r_[leaf, leaf[1:], np.roll(leaf, 1)]
    g = graphgen.from_edges(leaves + 2, src, dst, symmetrize=True)
    w = graphgen.weights(g, seed=leaves, lo=1, hi=top)
    roots = [0, 1, 2, leaves // 2, leaves + 1]
    for tuning in ({**BUCKETS, "hub_min_deg": 1024, "block_min_deg": 512}, {**BUCKETS, "sssp_delta": 2}):
        dist = gpu.sssp(load(gpu, g, w, tuning), roots).cpu().numpy()
        for i, r in enumerate(roots):
            assert np.array_equal(dist[i], oracle.sssp(g.offsets, g.cols, w, r)), (tuning, r)


def test_bucket_sssp_same_partition_again(gpu):
    """More roots than the scratch was made for, then fewer."""
    rng = np.random.default_rng(5)
    n = 3000
    g = graphgen.from_edges(n, rng.integers(0, n, 4 * n), rng.integers(0, n, 4 * n), symmetrize=True)
    w = graphgen.weights(g, seed=1)
    P = load(gpu, g, w, BUCKETS)
    for count in (1, 3, 8, 20, 2):
        roots = rng.integers(0, n, count).tolist()
        dist = gpu.sssp(P, roots).cpu().numpy()
        for i, r in enumerate(roots):
            assert np.array_equal(dist[i], oracle.sssp(g.offsets, g.cols, w, r)), (count, i)


# ---------------------------------------- messages of the hybrid split

@pytest.mark.parametrize("n,alpha", [(40, 0.3), (300, 0.5), (4001, 0.5), (120000, 0.7)])
def test_hybrid_messages_of_each_size(gpu, n, alpha):
    """Messages of a few words, with a tail past their last 16 bytes, of more
    than one block, and (the largest: over 2^15 host vertices) by copies."""
    rng = np.random.default_rng(n)
    g = graphgen.from_edges(n, rng.integers(0, n, 4 * n), rng.integers(0, n, 4 * n), symmetrize=True)
    G = gpu.graph_load_csr(g.n, g.offsets, g.cols, None, symmetric=True)
    P = gpu.partition_by_degree(G, "high", alpha, seed=3)
    if n == 120000:
        assert gpu.partition_info(P)["cpu_vertices"] * 4 > 1 << 17
    roots = [0, n // 2, n - 1]
    lev = gpu.bfs(P, roots).cpu().numpy()
    for i, r in enumerate(roots):
        assert np.array_equal(lev[i], oracle.bfs(g.offsets, g.cols, r)), r
    # per iteration the rounding of a rank's contributions, and of what the
    # sums of one side become on the way to the other
    iters = 5
    want = oracle.pagerank(g.offsets, g.cols, iterations=iters)
    r = gpu.pagerank(P, iterations=iters).cpu().numpy().astype(np.float64)
    assert np.all(np.abs(r - want) <= (2 * iters + 2) * 2.0**-24 * want)


# ---------------------- betweenness rows shared by several blocks

@pytest.mark.parametrize("rows", [1, 511, 512, 513, 1024, 1025])
@pytest.mark.parametrize("deg", [16, 64, 300])
def test_betweenness_rows_shared_or_not(gpu, rows, deg):
    """`rows` vertices of equal degree, at and past the most that are shared,
    in the WAVE, BLOCK and HUB bin, with room in the partial sums for many,
    few and (16 edges a row) not all of them; sources on both sides."""
    rng = np.random.default_rng(rows + deg)
    pool = max(2 * deg, 400)
    cols = np.concatenate([rng.choice(pool, deg, replace=False) for _ in range(rows)])
    src = np.repeat(pool + np.arange(rows), deg)
    # the pool hangs together by a ring (levels of several vertices each)
    g = graphgen.from_edges(pool + rows, np.r_[src, np.arange(pool)], np.r_[cols, (np.arange(pool) + 1) % pool],
                            symmetrize=True)
    srcs = [0, pool // 3, pool, pool + rows - 1]
    ref = oracle.bc(g.offsets, g.cols, srcs)
    bins = {"g4_min_deg": 2, "g16_min_deg": 4, "wave_min_deg": 8, "block_min_deg": 50, "hub_min_deg": 200}
    for f in (gpu.bc, gpu.bc_batched):
        got = f(load(gpu, g, None, bins), srcs).cpu().numpy().astype(np.float64)
        assert np.all(np.abs(got - ref) <= 1e-5 * np.abs(ref) + 1e-6 * max(ref.max(), 1.0))


@pytest.mark.parametrize("rows,deg", [(1, 16), (513, 16), (1, 300), (512, 64), (1025, 300)])
def test_betweenness_of_one_source(gpu, rows, deg):
    """The same rows for a source at a time: long ones of each bin and rows
    past the most that are shared, added up over the calls."""
    rng = np.random.default_rng(rows + deg)
    pool = max(2 * deg, 400)
    cols = np.concatenate([rng.choice(pool, deg, replace=False) for _ in range(rows)])
    src = np.repeat(pool + np.arange(rows), deg)
    g = graphgen.from_edges(pool + rows, np.r_[src, np.arange(pool)], np.r_[cols, (np.arange(pool) + 1) % pool],
                            symmetrize=True)
    bins = {"g4_min_deg": 2, "g16_min_deg": 4, "wave_min_deg": 8, "block_min_deg": 50, "hub_min_deg": 200,
            "hub_chunk": 256}
    P = load(gpu, g, None, bins)
    for s in (0, pool // 3, pool, pool + rows - 1):
        ref = oracle.bc(g.offsets, g.cols, [s])
        got = gpu.bc(P, [s]).cpu().numpy().astype(np.float64)
        assert np.all(np.abs(got - ref) <= 1e-5 * np.abs(ref) + 1e-6 * max(ref.max(), 1.0)), s


@pytest.mark.parametrize("n,count", [(65535, 1), (65536, 2), (131072, 2), (131072, 3), (300000, 4), (300000, 5)])
def test_routes_with_edges_in_host_memory(gpu, n, count):
    """Roots on either side of one per 65,536 vertices, and SSSP on either
    side of 2^18 vertices."""
    rng = np.random.default_rng(n + count)
    g = graphgen.from_edges(n, rng.integers(0, n, 3 * n), rng.integers(0, n, 3 * n), symmetrize=True)
    w = graphgen.weights(g, seed=2)
    P = load(gpu, g, w, {"mapped_edges": 1})
    roots = rng.integers(0, n, count).tolist()
    lev, dist = gpu.bfs(P, roots).cpu().numpy(), gpu.sssp(P, roots[:2]).cpu().numpy()
    for i, r in enumerate(roots):
        assert np.array_equal(lev[i], oracle.bfs(g.offsets, g.cols, r)), i
        if i < 2:
            assert np.array_equal(dist[i], oracle.sssp(g.offsets, g.cols, w, r)), i
