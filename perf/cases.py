"""Timed workloads of the library, each through its Python entry points.

Graphs are seeded synthetic inputs made on the GPU: R-MAT with the
parameters (0.57, 0.19, 0.19, 0.05) and 16 generated edges per vertex, or
uniform G(n, 4n), with self-loops and duplicates dropped, ids permuted and,
where a case is symmetric, both directions of every edge.  Weights are
int32 in [1, 255], equal for both directions of an edge.

`listed()` and `draw()` name the workloads, `prepare()` makes the graph, its
partition, the roots and the output buffers, `run()` makes one call, `exact()`
gives floating results in 64 bits, `work()` the bytes and operations a call
cannot do without.
"""
import math

import numpy as np
import torch

import paper_1312_3018_amd as tg

A, B, C = 0.57, 0.19, 0.19

# Per operation: the range of vertex counts, of roots (or iterations), and the
# most vertices x roots (or edges x iterations, in vertices) of one call.
RANGES = {
    "bfs": (1 << 12, 1 << 22, 1, 32),
    "bfs_batched": (1 << 14, 1 << 20, 8, 64),
    "sssp": (1 << 12, 1 << 22, 1, 8),
    "sssp_batched": (1 << 12, 1 << 18, 8, 64),
    "pagerank": (1 << 12, 1 << 22, 5, 20),
    "cc": (1 << 12, 1 << 21, 1, 1),
    "bc": (1 << 12, 1 << 18, 1, 4),
    "bc_batched": (1 << 12, 1 << 20, 16, 64),
    "hybrid": (1 << 16, 1 << 20, 1, 4),
}


def listed():
    return [
        # one breadth-first search with its tree on a small graph: a single
        # interactive query, bound by launches and waits
        {"name": "bfs_one", "op": "bfs", "graph": "rmat", "vertices": 1 << 14, "symmetric": True, "count": 1,
         "parents": True},
        # many searches over a large scale-free graph: the benchmark's BFS part
        {"name": "bfs_many", "op": "bfs", "graph": "rmat", "vertices": 1 << 22, "symmetric": True, "count": 32,
         "parents": False},
        # 64 searches at once on a uniform graph, as the query server's slots run them
        {"name": "bfs_batch", "op": "bfs_batched", "graph": "uniform", "vertices": 1000003, "symmetric": True,
         "count": 64},
        # one shortest-path query on a small directed graph
        {"name": "sssp_one", "op": "sssp", "graph": "rmat", "vertices": 50021, "symmetric": False, "count": 1},
        # several shortest-path searches over a large graph: the benchmark's SSSP part
        {"name": "sssp_many", "op": "sssp", "graph": "rmat", "vertices": 1 << 22, "symmetric": True, "count": 8},
        # 64 shortest-path queries at once, as the query server's slots run them
        {"name": "sssp_batch", "op": "sssp_batched", "graph": "rmat", "vertices": 1 << 18, "symmetric": True,
         "count": 64},
        # ranking of a small directed graph, dangling mass discarded
        {"name": "pagerank_small", "op": "pagerank", "graph": "rmat", "vertices": 30011, "symmetric": False,
         "count": 20, "dangling": "drop"},
        # ranking of a large graph: the benchmark's PageRank part
        {"name": "pagerank_large", "op": "pagerank", "graph": "rmat", "vertices": 1 << 22, "symmetric": True,
         "count": 20, "dangling": "uniform"},
        # weak components of a directed graph of ragged size
        {"name": "cc_directed", "op": "cc", "graph": "rmat", "vertices": 700001, "symmetric": False, "count": 1},
        # betweenness from a few sources, one at a time
        {"name": "bc_few", "op": "bc", "graph": "rmat", "vertices": 1 << 18, "symmetric": True, "count": 4},
        # betweenness from a sample of sources, 64 per chain (the betweenness benchmark)
        {"name": "bc_batch", "op": "bc_batched", "graph": "rmat", "vertices": 1 << 20, "symmetric": True, "count": 64},
        # the split between GPU and host threads: hubs holding a tenth of the
        # edges on the host, a few searches and ten PageRank iterations
        {"name": "hybrid_split", "op": "hybrid", "graph": "rmat", "vertices": 1 << 20, "symmetric": False,
         "count": 4},
    ]


def draw(rng):
    op = rng.choice(sorted(RANGES))
    lo, hi, clo, chi = RANGES[op]
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    case = {"op": op, "graph": "uniform" if op != "hybrid" and rng.random() < 0.25 else "rmat",
            "vertices": min(max(v, lo), hi), "symmetric": op != "hybrid" and rng.random() < 0.6,
            "count": rng.randint(clo, chi)}
    if op == "bfs":
        case["parents"] = case["vertices"] <= 1 << 16 and rng.random() < 0.5
    if op == "pagerank":
        case["dangling"] = rng.choice(["uniform", "drop"])
    return case


def _edges(case, gen):
    """(src, dst) of the generated edges, ids permuted, int64 on the GPU."""
    v = case["vertices"]
    if case["graph"] == "uniform":
        e = torch.randint(0, v, (2, 4 * v), generator=gen, device="cuda")
        return e[0], e[1]
    scale = max(1, (v - 1).bit_length())
    full = 1 << scale
    # edges of the next power of two, kept where both ends fall below v
    m = int(16 * v * (full / v) ** 2)
    src = torch.zeros(m, dtype=torch.int64, device="cuda")
    dst = torch.zeros(m, dtype=torch.int64, device="cuda")
    for _ in range(scale):
        u = torch.rand(m, generator=gen, device="cuda")
        low = u >= A + B
        src.mul_(2).add_(low)
        dst.mul_(2).add_(((u >= A) & ~low) | (u >= A + B + C))
    perm = torch.randperm(full, generator=gen, device="cuda")
    src, dst = perm[src], perm[dst]
    keep = (src < v) & (dst < v)
    return src[keep], dst[keep]


def _graph(case, seed):
    """CSR tensors (offsets int64, columns int32, weights int32) and the rows of the edges."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    v = case["vertices"]
    src, dst = _edges(case, gen)
    keep = src != dst
    src, dst = src[keep], dst[keep]
    if case["symmetric"]:
        src, dst = torch.cat([src, dst]), torch.cat([dst, src])
    key = torch.unique(src * v + dst)
    del src, dst
    row = torch.div(key, v, rounding_mode="floor")
    col = key - row * v
    off = torch.zeros(v + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(torch.bincount(row, minlength=v), 0, out=off[1:])
    # a weight per edge from its two ends (per unordered pair where symmetric)
    a, b = (torch.minimum(row, col), torch.maximum(row, col)) if case["symmetric"] else (row, col)
    h = (a * 1000003 + b * 7919 + int(seed) * 104729) & 0x7FFFFFFF
    h = (h * 48271 + 11) & 0x7FFFFFFF
    h = ((h ^ (h >> 15)) * 69621) & 0x7FFFFFFF
    w = (1 + (h >> 7) % 255).to(torch.int32)
    deg = off[1:] - off[:-1]
    cand = torch.nonzero(deg > 0).flatten()
    pick = torch.randperm(cand.numel(), generator=gen, device="cuda")[: case["count"]]
    roots = cand[pick].to(torch.int32).cpu().numpy()
    return off, col.to(torch.int32), w, row, roots


def prepare(case, seed):
    op, v = case["op"], case["vertices"]
    off, col, w, _, roots = _graph(case, seed)
    weighted = op in ("sssp", "sssp_batched")
    graph = tg.graph_load_csr(v, off, col, w if weighted else None, symmetric=case["symmetric"], validate=False)
    if op == "hybrid":
        part = tg.partition_by_degree(graph, "high", 0.1, seed=5)
    else:
        part = tg.partition_by_degree(graph)
    state = {"case": case, "part": part, "roots": roots}
    if op in ("pagerank", "bc", "bc_batched", "hybrid"):
        state["values"] = torch.empty(v, dtype=torch.float32, device="cuda")
    if op == "cc":
        state["rows"] = torch.empty(v, dtype=torch.int32, device="cuda")
    elif op not in ("pagerank", "bc", "bc_batched"):
        state["rows"] = torch.empty((len(roots), v), dtype=torch.int32, device="cuda")
    if case.get("parents"):
        state["parents"] = torch.empty((len(roots), v), dtype=torch.int32, device="cuda")
    return state


def run(state):
    case, part, roots = state["case"], state["part"], state["roots"]
    op = case["op"]
    if op == "bfs":
        if case["parents"]:
            return tg.bfs(part, roots, state["rows"], state["parents"])
        return tg.bfs(part, roots, state["rows"])
    if op == "bfs_batched":
        return tg.bfs_batched(part, roots, state["rows"])
    if op == "sssp":
        return tg.sssp(part, roots, state["rows"])
    if op == "sssp_batched":
        return tg.sssp_batched(part, roots, state["rows"])
    if op == "pagerank":
        return tg.pagerank(part, 0.85, case["count"], case["dangling"], state["values"])
    if op == "cc":
        return tg.cc(part, state["rows"])
    if op == "bc":
        return tg.bc(part, roots, state["values"])
    if op == "bc_batched":
        return tg.bc_batched(part, roots, state["values"])
    levels = tg.bfs(part, roots, state["rows"])
    return levels, tg.pagerank(part, 0.85, 10, "uniform", state["values"])


def _pagerank64(v, off, col, row, iterations, dangling):
    deg = (off[1:] - off[:-1]).double()
    r = torch.full((v,), 1.0 / v, dtype=torch.float64, device="cuda")
    for _ in range(iterations):
        c = torch.where(deg > 0, r / deg.clamp(min=1.0), torch.zeros_like(r))
        mass = float(r[deg == 0].sum()) if dangling == "uniform" else 0.0
        s = torch.zeros_like(r).index_add_(0, col, c[row])
        r = 0.15 / v + 0.85 * (s + mass / v)
    return r


def _gather_sum(x, keys, values, steps=1 << 22):
    """out[keys[e]] += x[values[e]] over rows of x, a bounded number of edges at a time."""
    out = torch.zeros_like(x)
    for e in range(0, keys.numel(), steps):
        out.index_add_(0, keys[e : e + steps], x[values[e : e + steps]])
    return out


def _bc64(v, col, row, sources):
    score = torch.zeros(v, dtype=torch.float64, device="cuda")
    for s0 in range(0, len(sources), 16):
        src = torch.from_numpy(sources[s0 : s0 + 16].astype(np.int64)).cuda()
        k = src.numel()
        at = torch.arange(k, device="cuda")
        sigma = torch.zeros((v, k), dtype=torch.float64, device="cuda")
        level = torch.full((v, k), -1, dtype=torch.int16, device="cuda")
        sigma[src, at] = 1.0
        level[src, at] = 0
        depth = 0
        while True:
            got = _gather_sum(torch.where(level == depth, sigma, 0.0), col, row)
            new = (level < 0) & (got > 0)
            if not bool(new.any()):
                break
            depth += 1
            sigma = torch.where(new, got, sigma)
            level[new] = depth
        delta = torch.zeros_like(sigma)
        for d in range(depth - 1, 0, -1):
            child = torch.where(level == d + 1, (1.0 + delta) / sigma.clamp(min=1.0), 0.0)
            delta = torch.where(level == d, sigma * _gather_sum(child, row, col), delta)
        score += delta.sum(1)
    return score


def exact(case, seed):
    op, v = case["op"], case["vertices"]
    if op not in ("pagerank", "bc", "bc_batched", "hybrid"):
        return None
    off, col, _, row, roots = _graph(case, seed)
    col = col.long()
    if op in ("bc", "bc_batched"):
        return _bc64(v, col, row, roots)
    if op == "pagerank":
        return _pagerank64(v, off, col, row, case["count"], case["dangling"])
    return None, _pagerank64(v, off, col, row, 10, "uniform")


def work(case):
    """Per call: the edges (4 bytes, 8 with weights) and offsets once, or once
    per iteration, and each output once; an addition and a product per edge
    where values are summed.  Edge counts are the expected ones before
    duplicates are dropped."""
    op, v, k = case["op"], case["vertices"], case["count"]
    e = (4 if case["graph"] == "uniform" else 16) * v * (2 if case["symmetric"] else 1)
    graph = 4 * e + 8 * (v + 1)
    if op in ("bfs", "bfs_batched"):
        return {"bytes": graph + 4 * v * k * (2 if case.get("parents") else 1), "flops": 0}
    if op in ("sssp", "sssp_batched"):
        return {"bytes": graph + 4 * e + 4 * v * k, "flops": 0}
    if op == "pagerank":
        return {"bytes": graph * k + 4 * v, "flops": 2 * e * k}
    if op == "cc":
        return {"bytes": graph + 4 * v, "flops": 0}
    if op in ("bc", "bc_batched"):
        return {"bytes": graph + 4 * v, "flops": 4 * e * k}
    return {"bytes": graph * 11 + 4 * v * (k + 1), "flops": 2 * e * 10}
