// Connected components (the fifth algorithm of section 9.4, run on the
// undirected graph): the label of a vertex is the smallest original id of its
// component; a directed graph gives its weak components.
//
// A forest of parent links over the local ids is grown by linking the two
// ends of an edge (the larger root is hooked under the smaller with a
// compare-and-swap) and flattened by compression, with a few neighbours per
// vertex first and the rest of the edges only where they can still matter
// (the neighbour sampling of Sutton, Ben-Nun and Barak, "Optimizing parallel
// graph connectivity computation via subgraph sampling", IPDPS 2018):
//   1. every vertex starts under its smallest sampled neighbour (local ids
//      are in decreasing-degree order, so that is a hub) and is compressed;
//   2. it is linked with its first four in-neighbours and compressed;
//   3. the most frequent root of a sample of vertices is taken as the large
//      component's, and only the vertices outside it link their remaining
//      edges -- in both directions on a directed graph, so that an edge with
//      one end inside is still seen from the other;
//   4. after the last compression each root takes the least original id of
//      its members, and every vertex its root's.
// A scale-free graph's large component is complete after step 2, so most
// edges are never read; what is left is bound by the random reads of the
// parent array (4 bytes a vertex, served by the L2) and by the launches.
// Minimum-label propagation over all edges, with atomic minima on the hubs,
// took 1.45 ms a call on R-MAT with 700,001 vertices and 10.6 M directed
// edges (1.04 ms of it in the pushes) and 8.9 ms on RMAT-24; this takes 0.094
// and 0.60 ms (26 M of RMAT-24's 521 M edges linked).
#include <algorithm>

#include "tg_internal.h"

using namespace tgk;

namespace {

constexpr int SAMPLE = 512;  // vertices sampled for the large component (one block)
constexpr int GIANT = 40;    // ws.counters: the large component's root

__device__ __forceinline__ int32_t fresh(const int32_t *comp, int32_t v) {
  return __hip_atomic_load(comp + v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Join the trees of a and b.  The first two reads may be old values: a
// former parent is still in the same tree.  Every further step replaces the
// larger of the two candidates by something smaller (the parent read for it
// or the value that beat the compare-and-swap), so the loop ends.
__device__ __forceinline__ void link(int32_t *comp, int32_t a, int32_t b) {
  int32_t p = comp[a], q = comp[b];
  while (p != q) {
    const int32_t hi = p > q ? p : q, lo = p > q ? q : p;
    int32_t up = fresh(comp, hi);
    if (up == hi) {
      up = atomicCAS(comp + hi, hi, lo);
      if (up == hi) return;
    }
    p = up;
    q = lo;
  }
}

__global__ __launch_bounds__(BLOCK) void k_cc_start(const int4 *__restrict__ head, const int64_t *__restrict__ off,
                                                    const int32_t *__restrict__ col, int directed, int64_t n,
                                                    int32_t *__restrict__ comp, int32_t *__restrict__ least) {
  const int64_t v = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (v >= n) return;
  int32_t c = (int32_t)v;
  const int32_t h = head[v].x;
  if (h >= 0) c = min(c, h);
  if (directed) {
    const int64_t e = off[v];
    if (e < off[v + 1]) c = min(c, col[e]);
  }
  comp[v] = c;
  least[v] = TG_INF;
}

// Every vertex directly under its root.  Each step halves the path with the
// value written at once, so that vertices further down the same path skip
// ahead; on a long path (many steps) the reads and writes go past the L2s,
// which do not see each other's writes within a launch.
__global__ __launch_bounds__(BLOCK) void k_cc_compress(int64_t n, int32_t *comp) {
  const int64_t v = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (v >= n) return;
  int32_t c = comp[v];
  for (int i = 0; i < 16; ++i) {
    const int32_t p = comp[c];
    if (p == c) return;
    comp[v] = c = p;
  }
  for (;;) {
    const int32_t p = fresh(comp, c);
    if (p == c) return;
    __hip_atomic_store(comp + v, p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    c = p;
  }
}

__global__ __launch_bounds__(BLOCK) void k_cc_link_head(const int4 *__restrict__ head, int64_t n, int32_t *comp,
                                                        unsigned long long *work) {
  const int64_t v = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  unsigned long long edges = 0;
  if (v < n) {
    const int4 h = head[v];
    const int32_t hu[4] = {h.x, h.y, h.z, h.w};
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (hu[k] >= 0) {
        link(comp, (int32_t)v, hu[k]);
        ++edges;
      }
  }
  edges = block_sum(edges);
  if (threadIdx.x == 0 && edges) stat_add(work, edges);
}

// One block: the most frequent root among SAMPLE vertices spread over [0, n).
__global__ __launch_bounds__(SAMPLE) void k_cc_giant(const int32_t *__restrict__ comp, int64_t n, uint32_t *giant) {
  __shared__ __align__(16) int32_t s[SAMPLE];
  __shared__ uint32_t best;
  const int t = threadIdx.x;
  s[t] = comp[n * t / SAMPLE];
  if (t == 0) best = 0u;
  __syncthreads();
  const int32_t mine = s[t];
  uint32_t count = 0;
  for (int i = 0; i < SAMPLE; i += 4) {
    const int4 x = *reinterpret_cast<const int4 *>(s + i);
    count += (x.x == mine ? 1u : 0u) + (x.y == mine ? 1u : 0u) + (x.z == mine ? 1u : 0u) + (x.w == mine ? 1u : 0u);
  }
  atomicMax(&best, (count << 16) | (uint32_t)t);
  __syncthreads();
  if (t == 0) *giant = (uint32_t)s[best & 0xFFFFu];
}

// The remaining edges [off[v] + skip, off[v + 1]) of the vertices of
// [v0, v1) outside the large component: one lane per vertex for short rows,
// the whole wave for long ones, one after another.
constexpr int SHORT_ROW = 8;
__global__ __launch_bounds__(BLOCK) void k_cc_link_rows(const int64_t *__restrict__ off,
                                                        const int32_t *__restrict__ col, int skip, int64_t v0,
                                                        int64_t v1, const uint32_t *__restrict__ giant, int32_t *comp,
                                                        unsigned long long *work) {
  const int lane = threadIdx.x & 63;
  const int64_t v = v0 + (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  int64_t e0 = 0, e1 = 0;
  if (v < v1 && comp[v] != (int32_t)*giant) {
    e0 = off[v] + skip;
    e1 = off[v + 1];
  }
  unsigned long long edges = e1 > e0 ? (unsigned long long)(e1 - e0) : 0ull;
  const bool wide = e1 - e0 > SHORT_ROW;
  if (!wide)
    for (int64_t e = e0; e < e1; ++e) link(comp, (int32_t)v, col[e]);
  for (uint64_t todo = __ballot(wide); todo; todo &= todo - 1) {
    const int src = __ffsll((long long)todo) - 1;
    const int64_t a0 = __shfl((long long)e0, src, 64), a1 = __shfl((long long)e1, src, 64);
    const int32_t row = __shfl((int32_t)v, src, 64);
    for (int64_t e = a0 + lane; e < a1; e += 64) link(comp, row, col[e]);
  }
  edges = block_sum(edges);
  if (threadIdx.x == 0 && edges) stat_add(work, edges);
}

// The same for the rows of [0, v1) of a symmetric graph's largest degrees:
// gridDim.y blocks share each row.
__global__ __launch_bounds__(BLOCK) void k_cc_link_hubs(const int64_t *__restrict__ off,
                                                        const int32_t *__restrict__ col, int skip, int64_t v1,
                                                        const uint32_t *__restrict__ giant, int32_t *comp,
                                                        unsigned long long *work) {
  const int32_t g = (int32_t)*giant;
  unsigned long long edges = 0;
  for (int64_t v = blockIdx.x; v < v1; v += gridDim.x) {
    // another block may move v's tree under the large component meanwhile:
    // the lanes that see it skip their edges, whose other ends are in the
    // large component too or link them from their own rows
    if (comp[v] == g) continue;
    const int64_t e1 = off[v + 1];
    for (int64_t e = off[v] + skip + (int64_t)blockIdx.y * BLOCK + threadIdx.x; e < e1;
         e += (int64_t)gridDim.y * BLOCK) {
      link(comp, (int32_t)v, col[e]);
      ++edges;
    }
  }
  edges = block_sum(edges);
  if (threadIdx.x == 0 && edges) stat_add(work, edges);
}

// least[root] = the smallest original id of the root's members.  A wave first
// folds the members of up to four of its roots, and the large component's
// members fold over the block's whole range, one atomic a block: atomics on
// one address take about 12 ns each (one a wave of 1024 blocks: 50 us).
__global__ __launch_bounds__(BLOCK) void k_cc_least(const int32_t *__restrict__ comp,
                                                    const int32_t *__restrict__ g_of_l, int64_t n,
                                                    const uint32_t *__restrict__ giant, int32_t *least) {
  const int lane = threadIdx.x & 63;
  const int32_t g = comp[*giant];
  int32_t fold = TG_INF;
  for (int64_t b = (int64_t)blockIdx.x * BLOCK; b < n; b += (int64_t)gridDim.x * BLOCK) {
    const int64_t v = b + threadIdx.x;
    const int32_t r = v < n ? comp[v] : -1;
    const int32_t id = v < n ? g_of_l[v] : TG_INF;
    if (r == g) fold = min(fold, id);
    uint64_t left = __ballot(r >= 0 && r != g);
    for (int k = 0; k < 4 && left; ++k) {
      const int lead = __ffsll((long long)left) - 1;
      const int32_t root = __shfl(r, lead, 64);
      const uint64_t same = __ballot(r == root);
      int32_t x = r == root ? id : TG_INF;
      if (same & (same - 1))  // wave-uniform: more than one member
        for (int o = 32; o > 0; o >>= 1) x = min(x, __shfl_xor(x, o, 64));
      if (lane == lead) atomicMin(least + root, x);
      left &= ~same;
    }
    if ((left >> lane) & 1ull) atomicMin(least + r, id);
  }
  __shared__ int32_t red[BLOCK / 64];
  for (int o = 32; o > 0; o >>= 1) fold = min(fold, __shfl_xor(fold, o, 64));
  if (lane == 0) red[threadIdx.x >> 6] = fold;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < BLOCK / 64; ++k) fold = min(fold, red[k]);
    if (fold < TG_INF) atomicMin(least + g, fold);
  }
}

__global__ __launch_bounds__(BLOCK) void k_cc_labels(const int32_t *__restrict__ comp,
                                                     const int32_t *__restrict__ least,
                                                     const int32_t *__restrict__ l_of_g, int64_t V,
                                                     int32_t *__restrict__ labels) {
  const int64_t gid = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (gid < V) labels[gid] = least[comp[l_of_g[gid]]];
}

}  // namespace

namespace tg {

// Labels (original ids) of the GPU partition's vertices.  The forest is in
// ws.state, the roots' least ids in ws.settled; spread counter 0 counts the
// edges linked.
int gpu_cc(tg_partition *p, int32_t *labels, hipStream_t s, int64_t *rounds_out) {
  GpuPart &g = p->gpu;
  Workspace &ws = p->ws;
  TG_TRY(ws.ensure(g, 0));
  if (rounds_out) *rounds_out = 0;
  if (g.n == 0) return TG_OK;
  const int64_t n = g.n;
  const dim3 nb((unsigned)((n + BLOCK - 1) / BLOCK)), tb(BLOCK);
  const int4 *head = reinterpret_cast<const int4 *>(g.in_head);
  const int directed = g.in_alias ? 0 : 1;
  int32_t *comp = ws.state, *least = ws.settled;
  uint32_t *giant = ws.counters + GIANT;
  hipLaunchKernelGGL(k_cc_start, nb, tb, 0, s, head, g.out.off, g.out.col, directed, n, comp, least);
  hipLaunchKernelGGL(k_cc_compress, nb, tb, 0, s, n, comp);
  const int tk = ktimer_start(s);
  hipLaunchKernelGGL(k_cc_link_head, nb, tb, 0, s, head, n, comp, ws.work);
  hipLaunchKernelGGL(k_cc_compress, nb, tb, 0, s, n, comp);
  // the large component is looked for among the vertices with edges, where
  // those are a prefix of the ids
  const int64_t nz = directed ? n : std::max<int64_t>(g.out_bins.bstart[BIN_ZERO], 1);
  hipLaunchKernelGGL(k_cc_giant, dim3(1), dim3(SAMPLE), 0, s, comp, nz, giant);
  // out-edges (a symmetric graph's head held its first four), then a
  // directed graph's in-edges past the head; the rows of 512 edges and more
  // (a prefix of the ids, by out-degree) are shared by several blocks each
  const int skip = directed ? 0 : 4;
  const int64_t big = g.out_bins.bstart[BIN_WAVE];
  if (big > 0)
    hipLaunchKernelGGL(k_cc_link_hubs, dim3((unsigned)std::min<int64_t>(big, 2048), 8), tb, 0, s, g.out.off,
                       g.out.col, skip, big, giant, comp, ws.work);
  if (nz > big)
    hipLaunchKernelGGL(k_cc_link_rows, dim3((unsigned)((nz - big + BLOCK - 1) / BLOCK)), tb, 0, s, g.out.off,
                       g.out.col, skip, big, nz, giant, comp, ws.work);
  if (directed)
    hipLaunchKernelGGL(k_cc_link_rows, nb, tb, 0, s, g.in.off, g.in.col, 4, (int64_t)0, n, giant, comp, ws.work);
  ktimer_stop(tk, s, "cc_push");
  hipLaunchKernelGGL(k_cc_compress, nb, tb, 0, s, n, comp);
  hipLaunchKernelGGL(k_cc_least, dim3(std::min(nb.x, 512u)), tb, 0, s, comp, g.g_of_l, n, giant, least);
  hipLaunchKernelGGL(k_cc_labels, dim3((unsigned)((g.n_global + BLOCK - 1) / BLOCK)), tb, 0, s, comp, least, g.l_of_g,
                     g.n_global, labels);
  TG_HIP(hipGetLastError());
  if (rounds_out) *rounds_out = 2;  // linking passes: the sampled edges, the rest
  return TG_OK;
}

}  // namespace tg
