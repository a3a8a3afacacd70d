// Searches whose cost is launches and waits, not edges: breadth-first search
// on small graphs, one workgroup per root in one launch, and shortest paths
// for a few roots, one launch per round for all of them.
#include <algorithm>
#include <memory>

#include "ms.h"

using namespace tgk;

namespace tg {
namespace {

// ------------------------------------------------------------------- BFS
//
// The whole search runs in one 1024-thread workgroup with its bitmaps and
// byte levels in LDS, so a level costs barriers and load latency (2-10 us)
// instead of four launches and a share of a host wait.  Top-down levels walk
// an LDS queue, a wave per vertex; bottom-up levels (Beamer's switch) give a
// lane to each unvisited vertex: its first four in-neighbours with one
// 16-byte load, twelve more from its row, then the wave takes the rows still
// open.  Many roots are as many workgroups.  RMAT-14, one root with parents:
// 298 us a call through the launched supersteps, 88 so; 64 roots: 419 in the
// 64-slot engine, 96 so.  (Four vertices per lane in flight in the bottom-up
// levels were slower, 114: the registers of 16 waves do not hold them.)
constexpr int BT = 1024;
constexpr int64_t SMALL_BFS_MAX_N = 65536;
constexpr int QMAX = 1024;      // largest frontier walked top-down
constexpr int MAX_BYTE = 254;   // deepest level kept in a byte

struct SmallBfsInfo {
  int32_t root, supersteps;  // local; out: -1: deeper than a byte holds
  u64 edges, vertices;       // expanded top-down
  u64 checked, examined;     // bottom-up, `steps` times
  int64_t steps;
};

struct SmallBfsArgs {
  const int64_t *off;
  const int32_t *col;
  const int32_t *ioff32;
  const int64_t *ioff64;
  const int32_t *icol;
  const int4 *head;
  const int32_t *l_of_g;
  int32_t *state;        // [roots][n] levels by local id
  int32_t *out;          // [roots][V] levels by original id
  SmallBfsInfo *info;    // [roots]
  int64_t n, V, m, n_in;
  int64_t alpha, beta;
  int do_switch;
};

// Lane-wide append of the lanes with `add` to the LDS queue.
__device__ __forceinline__ void push_lanes(bool add, int32_t v, int32_t *queue, uint32_t *count) {
  const uint64_t m = __ballot(add);
  if (!m) return;
  const int lane = threadIdx.x & 63;
  uint32_t base = 0;
  if (lane == __ffsll((long long)m) - 1) base = atomicAdd(count, (uint32_t)__popcll(m));
  base = __shfl(base, __ffsll((long long)m) - 1, 64);
  const uint32_t at = base + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
  if (add && at < QMAX) queue[at] = v;
}

__global__ __launch_bounds__(BT) void k_bfs_small(const SmallBfsArgs A) {
  extern __shared__ uint32_t lds[];
  const int W = (int)((A.n + 63) / 64) * 2;  // bitmap words: whole pairs
  uint32_t *vis = lds, *fr = vis + W, *nx = fr + W;
  int32_t *qa = reinterpret_cast<int32_t *>(nx + W), *qb = qa + QMAX;
  uint8_t *lev = reinterpret_cast<uint8_t *>(qb + QMAX);
  __shared__ uint32_t count;            // vertices that joined this superstep
  __shared__ unsigned long long edges;  // their out-degrees
  // of all levels, for the statistics: edges looked at bottom-up, vertices and
  // edges expanded top-down
  __shared__ unsigned long long looked, expanded, scanned;
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  SmallBfsInfo *info = A.info + blockIdx.x;
  const int32_t root = __builtin_amdgcn_readfirstlane(info->root);
  for (int i = t; i < W; i += BT) vis[i] = fr[i] = nx[i] = 0u;
  __syncthreads();
  if (t == 0) {
    vis[root >> 5] = fr[root >> 5] = 1u << (root & 31);
    lev[root] = 0;
    qa[0] = root;
    looked = expanded = scanned = 0ull;
  }
  int64_t m_u = A.m, m_f = A.off[root + 1] - A.off[root];
  int64_t n_f = 1;
  int L = 0, bu = 0;
  // vertices reached, and of the bottom-up levels the vertices that looked plus
  // 2^24 each (scalar registers are scarce here)
  int32_t reached = 1;
  uint32_t ups = 0;
  bool queued = true;  // qa holds the frontier
  for (;; ++L) {
    if (L >= MAX_BYTE) {
      if (t == 0) info->supersteps = -1;
      return;
    }
    m_u -= m_f;
    if (A.do_switch) {
      if (!bu && m_f > m_u / A.alpha) bu = 1;
      else if (bu && n_f < A.n / A.beta) bu = 0;
    }
    // a frontier beyond the queue can only be looked for (every level of a
    // graph without in-edges beyond the bottom-up rows would be empty)
    const bool up = bu || n_f > QMAX;
    if (up) ups += (1u << 24) + (uint32_t)max((int32_t)A.n_in - reached, 0);
    __syncthreads();
    if (t == 0) {
      count = 0u;
      edges = 0ull;
      if (!up) atomicAdd(&scanned, (unsigned long long)m_f);
    }
    if (!up && !queued) {
      // the queue of a frontier that a bottom-up level found
      __syncthreads();
      for (int i0 = wv * 64; i0 < W; i0 += BT) {
        uint32_t w = i0 + lane < W ? fr[i0 + lane] : 0u;
        while (__ballot(w != 0u)) {
          push_lanes(w != 0u, w ? (i0 + lane) * 32 + __ffs(w) - 1 : 0, qa, &count);
          w &= w - 1u;
        }
      }
      __syncthreads();
      if (t == 0) count = 0u;
    }
    __syncthreads();
    unsigned long long deg = 0;
    if (!up) {
      uint32_t rows = 0;
      for (int i = wv; i < (int)n_f; i += BT / 64) {
        const int32_t v = qa[i];
        const int64_t e0 = A.off[v], e1 = A.off[v + 1];
        rows += e1 > e0 ? 1u : 0u;
        for (int64_t e = e0; e < e1; e += 256) {
          int32_t nb[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) nb[k] = e + k * 64 + lane < e1 ? A.col[e + k * 64 + lane] : -1;
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            bool won = false;
            if (nb[k] >= 0) {
              const uint32_t bit = 1u << (nb[k] & 31);
              if (!(vis[nb[k] >> 5] & bit)) won = !(atomicOr(vis + (nb[k] >> 5), bit) & bit);
            }
            if (won) {
              atomicOr(nx + (nb[k] >> 5), 1u << (nb[k] & 31));
              lev[nb[k]] = (uint8_t)(L + 1);
              deg += (unsigned long long)(A.off[nb[k] + 1] - A.off[nb[k]]);
            }
            push_lanes(won, nb[k], qb, &count);
          }
        }
      }
      if (lane == 0 && rows) atomicAdd(&expanded, (unsigned long long)rows);
    } else {
      uint32_t joined = 0, checked = 0;
      int64_t walked = 0;
      const auto in = [&](int32_t u) { return u >= 0 && ((fr[u >> 5] >> (u & 31)) & 1u); };
      for (int64_t v0 = wv * 64; v0 < A.n_in; v0 += BT) {
        const int64_t v = v0 + lane;
        const bool open = v < A.n_in && !((vis[v >> 5] >> (v & 31)) & 1u);
        bool hit = false;
        int64_t e = 0, e1 = 0;
        if (open) {
          const int4 h = A.head[v];
          hit = in(h.x) || in(h.y) || in(h.z) || in(h.w);
          // (ids of a short row end in -1)
          checked += (uint32_t)(4 + (h.x >> 31) + (h.y >> 31) + (h.z >> 31) + (h.w >> 31));
          if (!hit && h.w >= 0) {
            e = (A.ioff32 ? (int64_t)A.ioff32[v] : A.ioff64[v]) + 4;
            e1 = A.ioff32 ? (int64_t)A.ioff32[v + 1] : A.ioff64[v + 1];
            for (int r = 0; r < 3 && e < e1 && !hit; ++r, e += 4) {
              int32_t u[4];
#pragma unroll
              for (int k = 0; k < 4; ++k) u[k] = A.icol[e + k < e1 ? e + k : e1 - 1];
              hit = in(u[0]) || in(u[1]) || in(u[2]) || in(u[3]);
              checked += (uint32_t)min(e1 - e, (int64_t)4);
            }
          }
        }
        for (uint64_t todo = __ballot(!hit && e < e1); todo; todo &= todo - 1) {
          const int src = __ffsll((long long)todo) - 1;
          const int64_t a1 = lane_i64(e1, src);
          bool found = false;
          for (int64_t b = lane_i64(e, src); b < a1 && !found; b += 256) {
            int32_t u[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) u[k] = b + k * 64 + lane < a1 ? A.icol[b + k * 64 + lane] : -1;
            found = __ballot(in(u[0]) || in(u[1]) || in(u[2]) || in(u[3])) != 0ull;
            walked += min(a1 - b, (int64_t)256);
          }
          if (lane == src) hit = found;
        }
        const uint64_t m = __ballot(hit);
        if (m) {
          // the wave's own two words
          if (lane == 0) nx[v0 >> 5] = (uint32_t)m;
          if (lane == 1) nx[(v0 >> 5) + 1] = (uint32_t)(m >> 32);
          joined += (uint32_t)__popcll(m);
          if (hit) {
            lev[v] = (uint8_t)(L + 1);
            deg += (unsigned long long)(A.off[v + 1] - A.off[v]);
          }
        }
      }
      const unsigned long long seen = (unsigned long long)wave_total(checked) + (unsigned long long)walked;
      if (lane == 0) {
        if (joined) atomicAdd(&count, joined);
        if (seen) atomicAdd(&looked, seen);
      }
    }
    deg = wave_sum(deg);
    if (lane == 0 && deg) atomicAdd(&edges, deg);
    __syncthreads();
    n_f = __builtin_amdgcn_readfirstlane((int)count);
    m_f = lane_i64((int64_t)edges, 0);
    reached += (int32_t)n_f;
    queued = !up;
    if (n_f == 0) break;
    for (int i = t; i < W; i += BT) {
      const uint32_t x = nx[i];
      fr[i] = x;
      nx[i] = 0u;
      if (up) vis[i] |= x;
    }
    int32_t *q = qa;
    qa = qb;
    qb = q;
  }
  // (the barrier above ordered every level written)
  int32_t *state = A.state + (int64_t)blockIdx.x * A.n;
  for (int64_t v = t; v < A.n; v += BT) state[v] = (vis[v >> 5] >> (v & 31)) & 1u ? (int32_t)lev[v] : TG_INF;
  int32_t *out = A.out + (int64_t)blockIdx.x * A.V;
  for (int32_t g0 = t; g0 < (int32_t)A.V; g0 += 8 * BT) {  // (eight ids in flight: 46.2 -> 44.9 us, RMAT-14)
    int32_t l[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) l[k] = g0 + k * BT < (int32_t)A.V ? A.l_of_g[g0 + k * BT] : 0;
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (g0 + k * BT < (int32_t)A.V) out[g0 + k * BT] = (vis[l[k] >> 5] >> (l[k] & 31)) & 1u ? (int32_t)lev[l[k]] : TG_INF;
  }
  if (t == 0) *info = SmallBfsInfo{root, L + 1, scanned, expanded, looked, ups & 0xFFFFFFu, ups >> 24};
}

size_t small_bfs_lds(int64_t n) {
  const size_t W = (size_t)((n + 63) / 64) * 2;
  return W * 3 * 4 + 2 * QMAX * 4 + (size_t)((n + 15) & ~(int64_t)15);
}

// ------------------------------------------------------------------ SSSP
//
// Frontier Bellman-Ford (section 7.3, Figure 20) with one launch per round
// and no queue: a vertex is active when its distance is below the one it
// last relaxed with, which its wave finds by reading both, and it relaxes
// its out-edges at once, in place.  A wave takes 1, 4 or 16 vertices by
// degree and walks the active ones' edges as one list, RT tiles of 64 in
// flight; rows of 512 edges and more get a 1024-thread block each.  Rounds
// are launched ahead in chunks; each leaves a flag if it found an active
// vertex, read once per chunk.  All roots of a call share the launches
// (grid y).  It relaxes 2-3 times the edges the buckets of the large-graph
// schedule do, in a quarter of the supersteps and with a sixth of the
// launches each.  R-MAT
// with 50,021 vertices, directed, one root: 2.53 ms through the buckets, 0.95
// in the 64-slot engine, 0.27 so; its widest round (44 us for 760,000 edges)
// is bound by the atomic minima.  (Gathering the minima of the 4,096 hottest
// vertices in LDS tables did not help: what the blocks flush is as much.)
constexpr int RT = 4;
constexpr int LIVE = 64;  // rounds a chunk holds at most
constexpr int ROUND_SLOTS = 256, ROUND_STRIDE = 16, ROUND_BITS = 36;

struct RoundArgs {
  const int64_t *off;
  const int32_t *col, *wgt;
  const uint32_t *cw;  // packed id | weight << 24, or null
  int32_t *dist, *settled;  // [roots][n]
  uint32_t *ovf;            // [roots][nwords]
  // [0]: some candidate did not fit; [1]: verdict; then two chunks of LIVE
  // flags, one per round
  uint32_t *flags;
  u64 *work;  // on ROUND_SLOTS lines: edges relaxed, and above ROUND_BITS the vertices they went out from
  int64_t n, nwords, hubs;
  RowSpans spans;
};

__global__ __launch_bounds__(BLOCK) void k_round_init(RoundArgs A, const int32_t *__restrict__ roots) {
  const int64_t y = blockIdx.y;
  const int32_t root = roots[y];
  for (int64_t v = (int64_t)blockIdx.x * BLOCK + threadIdx.x; v < A.n; v += (int64_t)gridDim.x * BLOCK) {
    A.dist[y * A.n + v] = v == root ? 0 : TG_INF;
    A.settled[y * A.n + v] = TG_INF;
    if (v < A.nwords) A.ovf[y * A.nwords + v] = 0u;
  }
  if (y == 0 && blockIdx.x == 0) {
    if (threadIdx.x < 3) A.flags[threadIdx.x] = 0u;
    for (int i = threadIdx.x; i < ROUND_SLOTS * ROUND_STRIDE; i += BLOCK) A.work[i] = 0ull;
  }
}

// sum: edges + vertices << ROUND_BITS
__device__ __forceinline__ void round_count(const RoundArgs &A, u64 sum) {
  atomicAdd(A.work + (size_t)(blockIdx.x % ROUND_SLOTS) * ROUND_STRIDE, sum);
}

__device__ __forceinline__ void round_relax(const RoundArgs &A, int32_t *dist, uint32_t *ovf, int32_t dv, int32_t nb,
                                            int32_t wt, int32_t cur) {
  // below 2^32: both are below 2^31
  const uint32_t nd = (uint32_t)dv + (uint32_t)wt;
  if (nd >= (uint32_t)TG_INF) {
    // cannot improve a finite distance; matters only if nb stays unreached
    if (cur == TG_INF) {
      atomicOr(ovf + (nb >> 5), 1u << (nb & 31));
      A.flags[0] = 1u;
    }
  } else if ((int32_t)nd < cur) {
    atomicMin(dist + nb, (int32_t)nd);  // no return value: nothing waits on it
  }
}

// (plain loads: the next rounds read the same edges, which fit the caches)
__device__ __forceinline__ void round_edge(const RoundArgs &A, int64_t e, int32_t &nb, int32_t &wt) {
  if (A.cw) {
    const uint32_t x = A.cw[e];
    nb = (int32_t)(x & 0xFFFFFFu);
    wt = (int32_t)(x >> 24);
  } else {
    nb = A.col[e];
    wt = A.wgt[e];
  }
}

constexpr int RB = 1024;
__global__ __launch_bounds__(RB) void k_round(const RoundArgs A, int live, int live_next) {
  const int64_t y = blockIdx.y;
  int32_t *dist = A.dist + y * A.n, *settled = A.settled + y * A.n;
  uint32_t *ovf = A.ovf + y * A.nwords;
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  if (blockIdx.x == 0 && y == 0 && t == 0) A.flags[live_next] = 0u;  // the next round's
  if ((int64_t)blockIdx.x < A.hubs) {
    const int64_t v = blockIdx.x;
    __shared__ int32_t sd;
    if (t == 0) {
      // one reader: every wave relaxes with the value noted as settled
      const int32_t d = dist[v];
      sd = d < settled[v] ? d : -1;
      if (sd >= 0) {
        settled[v] = d;
        A.flags[live] = 1u;
      }
    }
    __syncthreads();
    const int32_t dv = sd;
    if (dv < 0) return;
    const int64_t e1 = A.off[v + 1];
    for (int64_t e = A.off[v] + t; e < e1; e += RT * RB) {
      int32_t nb[RT], wt[RT], cur[RT];
#pragma unroll
      for (int q = 0; q < RT; ++q) {
        nb[q] = -1;
        if (e + q * RB < e1) round_edge(A, e + q * RB, nb[q], wt[q]);
      }
#pragma unroll
      for (int q = 0; q < RT; ++q) cur[q] = nb[q] >= 0 ? dist[nb[q]] : 0;
#pragma unroll
      for (int q = 0; q < RT; ++q)
        if (nb[q] >= 0) round_relax(A, dist, ovf, dv, nb[q], wt[q], cur[q]);
    }
    if (t == 0) round_count(A, (u64)(e1 - A.off[v]) + (1ull << ROUND_BITS));
    return;
  }
  u64 relaxed = 0;
  const int64_t wave = ((int64_t)blockIdx.x - A.hubs) * (RB / 64) + wv;
  const int64_t waves = ((int64_t)gridDim.x - A.hubs) * (RB / 64);
  for_row_spans(A.spans, wave, waves, [&](int64_t i, int k) {
    Entries E;
    // the mask holds the distance an active vertex relaxes with
    E.load([](int64_t x) { return (int32_t)x; },
           [&](int64_t, int32_t v) -> u64 {
             const int32_t d = dist[v];
             if (d >= settled[v]) return 0ull;
             settled[v] = d;
             return (1ull << 32) | (u64)(uint32_t)d;
           },
           i, k, A.off);
    const u64 on = __ballot(E.m != 0ull);
    if (!on) return;
    if (lane == 0) A.flags[live] = 1u;
    // (rows of these spans are below the BLOCK bin's degree: the list fits 32 bits)
    const int32_t len = (int32_t)E.total;
    for (int32_t t0 = 0; t0 < len; t0 += 64 * RT) {
      int32_t nb[RT], wt[RT], cur[RT], dv[RT];
#pragma unroll
      for (int q = 0; q < RT; ++q) {
        const int32_t p = t0 + q * 64 + lane;
        const int own = E.owner(p);
        const int64_t e = __shfl((long long)E.e0, own, 64) + (p - __shfl(E.start, own, 64));
        dv[q] = __shfl((int32_t)(uint32_t)E.m, own, 64);
        nb[q] = -1;
        if (p < len) round_edge(A, e, nb[q], wt[q]);
      }
#pragma unroll
      for (int q = 0; q < RT; ++q) cur[q] = nb[q] >= 0 ? dist[nb[q]] : 0;
#pragma unroll
      for (int q = 0; q < RT; ++q)
        if (nb[q] >= 0) round_relax(A, dist, ovf, dv[q], nb[q], wt[q], cur[q]);
    }
    relaxed += (u64)E.total + ((u64)__popcll(on) << ROUND_BITS);
  });
  // (last: a later read would wait for the addition)
  if (lane == 0 && relaxed) round_count(A, relaxed);
}

// flags[1] = 1 if some vertex with an overflowing candidate stayed unreached.
__global__ __launch_bounds__(BLOCK) void k_round_verdict(RoundArgs A) {
  const int64_t y = blockIdx.y, v = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (v < A.n && ((A.ovf[y * A.nwords + (v >> 5)] >> (v & 31)) & 1u) && A.dist[y * A.n + v] == TG_INF)
    A.flags[1] = 1u;
}

// (The first block leaves the counters' sums in pinned memory: their lines are
// slow to read from the host.)
__global__ __launch_bounds__(BLOCK) void k_round_collect(const int32_t *__restrict__ l_of_g,
                                                         const int32_t *__restrict__ dist, int64_t n, int64_t V,
                                                         int32_t *__restrict__ out, const u64 *work, u64 *sums) {
  static_assert(ROUND_SLOTS == BLOCK, "a counter a thread");
  const int64_t y = blockIdx.y, gid = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (blockIdx.x == 0 && y == 0) {
    const u64 x = work[(size_t)threadIdx.x * ROUND_STRIDE];
    const u64 edges = block_sum(x & ((1ull << ROUND_BITS) - 1)), verts = block_sum(x >> ROUND_BITS);
    if (threadIdx.x == 0) {
      sums[0] = edges;
      sums[1] = verts;
    }
  }
  if (gid < V) out[y * V + gid] = dist[y * n + l_of_g[gid]];
}

}  // namespace

// Scratch of both searches (lazy, per partition): per root a row of vertex
// state, and a few words per root.
struct SmallState {
  DevArena arena;
  int64_t rows = 0;  // entries of `state`
  int32_t *state = nullptr;
  uint32_t *flags = nullptr, *h_flags = nullptr;
  u64 *work = nullptr, *h_work = nullptr;  // the rounds' counters; their sums
  int32_t *roots = nullptr;
  SmallBfsInfo *info = nullptr;
  int32_t *h_roots = nullptr;
  SmallBfsInfo *h_info = nullptr;
  ~SmallState() {
    if (h_roots) TG_QUIET(hipHostFree(h_roots));
    if (h_info) TG_QUIET(hipHostFree(h_info));
    if (h_flags) TG_QUIET(hipHostFree(h_flags));
    if (h_work) TG_QUIET(hipHostFree(h_work));
  }
};

void small_free(tg_partition *p) {
  delete p->small;
  p->small = nullptr;
}

namespace {

constexpr int64_t CHUNK = 64;  // roots per launch

template <typename T>
int pinned(T **p, size_t count) {
  if (hipHostMalloc((void **)p, count * sizeof(T), hipHostMallocDefault) == hipSuccess) return TG_OK;
  (void)hipGetLastError();
  *p = nullptr;
  return set_error(TG_ENOMEM, "hipHostMalloc(%zu bytes) failed", count * sizeof(T));
}

int small_state(tg_partition *p, int64_t rows, SmallState **out) {
  if (!p->small) {
    // (kept only when whole)
    std::unique_ptr<SmallState> made(new (std::nothrow) SmallState());
    if (!made) return set_error(TG_ENOMEM, "out of host memory");
    TG_TRY(dalloc(made->arena, &made->roots, (size_t)CHUNK));
    TG_TRY(dalloc(made->arena, &made->info, (size_t)CHUNK));
    TG_TRY(dalloc(made->arena, &made->flags, (size_t)(2 + 2 * LIVE)));
    TG_TRY(dalloc(made->arena, &made->work, (size_t)ROUND_SLOTS * ROUND_STRIDE));
    TG_TRY(pinned(&made->h_flags, (size_t)(2 + 2 * LIVE)));
    TG_TRY(pinned(&made->h_work, (size_t)2));
    TG_TRY(pinned(&made->h_roots, (size_t)CHUNK));
    TG_TRY(pinned(&made->h_info, (size_t)CHUNK));
    p->small = made.release();
  }
  SmallState &S = *p->small;
  if (S.rows < rows) {
    if (S.state) S.arena.release_one(S.state);
    S.state = nullptr;
    S.rows = 0;
    TG_TRY(dalloc(S.arena, &S.state, (size_t)rows));
    S.rows = rows;
  }
  *out = &S;
  return TG_OK;
}

}  // namespace

// (us, launched single search or engine, whichever is less / one workgroup
// per root, 1 and 64 roots: R-MAT 2^12 221, 400 / 51, 51; 2^14 189, 419 / 84,
// 96; 2^16 189, 584 / 186, 224; uniform 2^13 240, 328 / 92, 104; 2^16 296, 441
// / 385, 434: without hubs most rows are read to their end, and one CU is too
// few for them.)
bool small_bfs_supported(const GpuPart &g) {
  if (g.n <= 0 || small_bfs_lds(g.n) > (size_t)rows_lds_limit()) return false;
  const bool hubs = g.h_deg[0] * g.n >= 16 * g.m;  // largest degree at least 16 times the mean
  return g.n <= (hubs ? SMALL_BFS_MAX_N : SMALL_BFS_MAX_N / 2);
}

int small_bfs(tg_partition *p, const int32_t *roots, int32_t nr, int32_t *levels, int32_t *parents, hipStream_t s,
              int64_t *supersteps, SearchWork *work, bool *deep) {
  const GpuPart &g = p->gpu;
  const Tuning &t = p->tune;
  SmallState *S = nullptr;
  TG_TRY(small_state(p, std::min<int64_t>(nr, CHUNK) * g.n, &S));
  *deep = false;
  for (int64_t c0 = 0; c0 < nr; c0 += CHUNK) {
    const int64_t cn = std::min<int64_t>(CHUNK, nr - c0);
    for (int64_t k = 0; k < cn; ++k) {
      S->h_roots[k] = p->h_l_of_g[roots[c0 + k]];
      S->h_info[k] = SmallBfsInfo{S->h_roots[k], 0, 0, 0, 0, 0, 0};
    }
    TG_HIP(hipMemcpyAsync(S->info, S->h_info, (size_t)cn * sizeof(SmallBfsInfo), hipMemcpyHostToDevice, s));
    SmallBfsArgs A{g.out.off, g.out.col, g.in_off32, g.in.off, g.in.col, reinterpret_cast<const int4 *>(g.in_head),
                   g.l_of_g, S->state, levels + c0 * g.n_global, S->info, g.n, g.n_global, g.m,
                   g.in_alias ? g.out_bins.bstart[BIN_ZERO] : g.n, t.bfs_alpha, t.bfs_beta, (int)t.bfs_do};
    const int tk = ktimer_start(s);
    hipLaunchKernelGGL(k_bfs_small, dim3((unsigned)cn), dim3(BT), small_bfs_lds(g.n), s, A);
    ktimer_stop(tk, s, "bfs_small");
    TG_HIP(hipGetLastError());
    if (parents)
      for (int64_t k = 0; k < cn; ++k)
        TG_TRY(bfs_parents(g, nullptr, S->state + k * g.n, S->h_roots[k], parents + (c0 + k) * g.n_global, s));
    TG_HIP(hipMemcpyAsync(S->h_info, S->info, (size_t)cn * sizeof(SmallBfsInfo), hipMemcpyDeviceToHost, s));
    TG_HIP(hipStreamSynchronize(s));
    ktimer_flush();
    for (int64_t k = 0; k < cn; ++k) {
      const SmallBfsInfo &I = S->h_info[k];
      if (I.supersteps < 0) *deep = true;
      *supersteps += I.supersteps;
      work->edges += (double)I.edges;
      work->vertices += (double)I.vertices;
      work->checked += (double)I.checked;
      work->examined += (double)I.examined;
      work->steps += (double)I.steps;
    }
    if (*deep) return TG_OK;
  }
  work->lanes = (int)std::min<int64_t>(nr, CHUNK);
  return TG_OK;
}

int round_sssp(tg_partition *p, const int32_t *roots, int32_t nr, int32_t *dist, hipStream_t s, int64_t *rounds,
               SearchWork *work) {
  const GpuPart &g = p->gpu;
  const int64_t n = g.n, V = g.n_global, nwords = (n + 31) / 32;
  // roots per launch: as many as rows of 2^24 entries in all
  const int64_t per = std::max<int64_t>(1, std::min<int64_t>({(int64_t)nr, CHUNK, ((int64_t)1 << 24) / n}));
  SmallState *S = nullptr;
  TG_TRY(small_state(p, per * (2 * n + nwords), &S));
  for (int64_t c0 = 0; c0 < nr; c0 += per) {
    const int64_t cn = std::min<int64_t>(per, nr - c0);
    for (int64_t k = 0; k < cn; ++k) S->h_roots[k] = p->h_l_of_g[roots[c0 + k]];
    TG_HIP(hipMemcpyAsync(S->roots, S->h_roots, (size_t)cn * sizeof(int32_t), hipMemcpyHostToDevice, s));
    RoundArgs A{g.out.off, g.out.col, g.out.w, p->tune.sssp_packed ? g.out.cw : nullptr, S->state, S->state + per * n,
                reinterpret_cast<uint32_t *>(S->state + 2 * per * n), S->flags,
                S->work, n, nwords,
                // (rows past 2^31 / 1024 blocks would not fit the grid: the waves take any row)
                std::min<int64_t>(g.out_bins.bstart[BIN_WAVE], 1 << 20), {}};
    A.spans = RowSpans{A.hubs, std::max(A.hubs, g.out_bins.bstart[BIN_G16]), std::max(A.hubs, g.out_bins.bstart[BIN_G4]),
                       std::max(A.hubs, g.out_bins.bstart[BIN_ZERO])};
    const unsigned y = (unsigned)cn;
    hipLaunchKernelGGL(k_round_init, dim3((unsigned)std::min<int64_t>((n + BLOCK - 1) / BLOCK, 4096), y), dim3(BLOCK), 0,
                       s, A, S->roots);
    const unsigned grid = (unsigned)(A.hubs + std::min<int64_t>((A.spans.waves() + RB / 64 - 1) / (RB / 64), 16384));
    int64_t done = 0;
    int half = 0;
    for (int chunk = 12;; chunk = std::min(done < 32 ? 4 : (int)(done / 2), LIVE - 1), half ^= 1) {
      // a frontier Bellman-Ford settles within |V| rounds
      if (done > n + LIVE) return set_error(TG_EDEVICE, "sssp: no convergence after %lld rounds", (long long)done);
      const int f0 = 2 + half * LIVE, f1 = 2 + (half ^ 1) * LIVE;
      const int tk = ktimer_start(s);
      for (int k = 0; k < chunk && grid > 0; ++k)
        hipLaunchKernelGGL(k_round, dim3(grid, y), dim3(RB), 0, s, A, f0 + k, k + 1 < chunk ? f0 + k + 1 : f1);
      ktimer_stop(tk, s, "sssp_round");
      TG_HIP(hipGetLastError());
      TG_HIP(hipMemcpyAsync(S->h_flags, S->flags, (2 + 2 * LIVE) * sizeof(uint32_t), hipMemcpyDeviceToHost, s));
      TG_HIP(hipStreamSynchronize(s));
      ktimer_flush();
      int k = 0;
      while (k < chunk && grid > 0 && S->h_flags[f0 + k]) ++k;
      done += k;
      if (k < chunk) break;  // a round without an active vertex
    }
    *rounds += done;
    if (S->h_flags[0]) {
      hipLaunchKernelGGL(k_round_verdict, dim3((unsigned)((n + BLOCK - 1) / BLOCK), y), dim3(BLOCK), 0, s, A);
      TG_HIP(hipMemcpyAsync(S->h_flags, S->flags, 2 * sizeof(uint32_t), hipMemcpyDeviceToHost, s));
      TG_HIP(hipStreamSynchronize(s));
      if (S->h_flags[1]) return set_error(TG_ERANGE, "sssp: a shortest-path distance does not fit below INT32_MAX");
    }
    hipLaunchKernelGGL(k_round_collect, dim3((unsigned)((V + BLOCK - 1) / BLOCK), y), dim3(BLOCK), 0, s, g.l_of_g,
                       S->state, n, V, dist + c0 * V, S->work, S->h_work);
    TG_HIP(hipGetLastError());
    TG_HIP(hipStreamSynchronize(s));
    work->edges += (double)S->h_work[0];
    work->vertices += (double)S->h_work[1];
  }
  work->lanes = (int)per;
  return TG_OK;
}

}  // namespace tg
