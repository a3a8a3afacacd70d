// Multi-source supersteps shared by the slot engine (slots.hip) and batched
// betweenness (bcb.hip): up to 64 searches advance together, one bit per
// search ("slot") in a vertex's frontier, visited and next masks.
//
// Every slot takes its own direction each superstep.  A slot whose frontier
// holds many edges is pulled: every vertex it has not visited looks through
// its in-neighbours' frontier masks and stops once every pulled slot it
// still wants is found.  The other slots are pushed along the frontier's
// out-edges.  (One direction for all would not do: a slot that lags behind,
// its frontier still small, is wanted by nearly every vertex and found by
// few, so that no row's scan could stop early.)
#pragma once
#include "tg_internal.h"

namespace tg {

using u64 = unsigned long long;
constexpr int kSlots = 64;

// Device state of a chain of supersteps, read back once per superstep.
// Per-slot sums are kept in MF_COPIES copies (block b adds to copy b mod
// MF_COPIES, the host adds them up): atomics on one address take about 12 ns
// each.
constexpr int MF_COPIES = 8;
struct MsState {
  Plan plan;
  // BFS: per slot, the edges of its frontier plus its vertices (0: no
  // frontier).  SSSP: [.][c][0] the OR of the frontier masks, [.][c][1] the
  // frontier's edges.  In turn: a superstep adds to one half and clears the
  // other.
  u64 mf[2][MF_COPIES][kSlots];
};
// Counters of a workspace's `work`.  BFS: (vertex, slot) pairs pushed and their
// edges; in-edges the pulls looked at and vertices that looked, each once for
// all slots.  SSSP: (vertex, slot) pairs of the frontiers and their edges.
enum { MS_PAIRS = 0, MS_EDGES = 1, MS_CHECKED = 2, MS_EXAMINED = 3, MS_COUNTERS = 4 };

// Slots of `alive` to pull: mf, the edges of the slot's frontier, against mu,
// those of the vertices it has not had on a frontier yet.
u64 ms_pull_slots(const u64 *mf, const int64_t *mu, u64 alive, const Tuning &t);
// Expand the frontier (masks `front`, queue and plan in ws, hp the host's
// copy of the plan) into next / ws.bits_a: slots of `pulled` by a pull, the
// rest of `alive` by a push.
int ms_expand(const GpuPart &g, Workspace &ws, const Tuning &t, const Plan &hp, const int32_t *queue,
              const u64 *front, const u64 *visited, u64 *next, u64 alive, u64 pulled, hipStream_t s);
// The pull of `pulled` for the vertices [0, hubs) alone (hub_rows(g) of
// them: a symmetric graph's rows of 512 edges and more) into next and (unless
// null) the bitmap `touched`, several waves a row.
int64_t hub_rows(const GpuPart &g);
int ms_pull_hubs(const GpuPart &g, Workspace &ws, uint32_t *touched, const u64 *front, const u64 *visited, u64 *next,
                 u64 pulled, hipStream_t s);

}  // namespace tg

namespace tgk {

using u64 = unsigned long long;

// Lane `src`'s 64-bit value, wave-uniform.
__device__ __forceinline__ u64 lane_mask(u64 m, int src) {
  return (u64)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)m, src) |
         ((u64)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(m >> 32), src) << 32);
}
__device__ __forceinline__ int64_t lane_i64(int64_t x, int src) { return (int64_t)lane_mask((u64)x, src); }

// Up to 64 queue entries held by one wave, lane j entry j, their edges
// walked as one list.
struct Entries {
  int32_t v;      // vertex
  u64 m;          // mask
  int64_t e0, d;  // first edge, number of edges
  int32_t start;  // first position in the list
  int64_t total;  // positions in the list (wave-uniform)
  int k, span;    // entries; the least power of two >= k

  template <class VertexF, class MaskF>
  __device__ __forceinline__ void load(VertexF vertex_of, MaskF mask_of, int64_t i0, int count, const int64_t *off) {
    const int lane = threadIdx.x & 63;
    k = count;
    v = 0;
    m = 0;
    e0 = d = 0;
    if (lane < k) {
      v = vertex_of(i0 + lane);
      m = mask_of(i0 + lane, v);
      e0 = off[v];
      if (m) d = off[v + 1] - e0;
    }
    int64_t inc = d;
    for (int o = 1; o < 64; o <<= 1) {
      const int64_t y = __shfl_up((long long)inc, o, 64);
      if (lane >= o) inc += y;
    }
    total = lane_i64(inc, 63);
    start = (int32_t)(inc - d);
    span = 1;
    while (span < k) span <<= 1;
  }
  // positions beyond 32 bits: the caller takes the entries one by one
  __device__ __forceinline__ bool long_list() const { return total >= ((int64_t)1 << 30); }
  // the entry that list position t falls in
  __device__ __forceinline__ int owner(int32_t t) const {
    int own = 0;
    for (int h = span >> 1; h > 0; h >>= 1) {
      const int32_t s = __shfl(start, own + h, 64);
      if (own + h < k && s <= t) own += h;
    }
    return own;
  }
};

// acc of lane s += weight of every lane whose mask has bit s.
__device__ __forceinline__ void add_by_slot(u64 nb, uint32_t weight, u64 &acc) {
  const int lane = threadIdx.x & 63;
  for (u64 todo = __ballot(nb != 0ull); todo; todo &= todo - 1) {
    const int j = __ffsll((long long)todo) - 1;
    const uint32_t w = (uint32_t)__builtin_amdgcn_readlane((int)weight, j);
    acc += (lane_mask(nb, j) >> lane) & 1ull ? (u64)w : 0ull;
  }
}

// The block's per-slot sums (block of THREADS) into its copy of mf, and the
// other half cleared for the next superstep.
template <int THREADS>
__device__ __forceinline__ void publish_by_slot(u64 acc, u64 (*mf)[tg::kSlots], u64 (*other)[tg::kSlots]) {
  __shared__ u64 red[THREADS];
  red[threadIdx.x] = acc;
  __syncthreads();
  if (threadIdx.x < 64) {
    u64 x = 0;
    for (int k = 0; k < THREADS / 64; ++k) x += red[k * 64 + threadIdx.x];
    if (x) atomicAdd(&mf[blockIdx.x % tg::MF_COPIES][threadIdx.x], x);
    if (blockIdx.x < tg::MF_COPIES) other[blockIdx.x][threadIdx.x] = 0ull;
    if (blockIdx.x == 0)
      for (int c = (int)gridDim.x; c < tg::MF_COPIES; ++c) other[c][threadIdx.x] = 0ull;
  }
}

// Rows of per-vertex state ([vertex][slot], lane = slot) combined along
// edges: for a row's neighbours u with mask[u] & m != 0, op.add(acc,
// op.load(u, mask), weight) in the row's order.  The ids, weights and masks
// of 64 edges are read at once, one per lane, edges that do not contribute
// are dropped, and FLY state rows are in flight together.
//   Op::X / A / P  a loaded row element, the accumulator, what begin() reads
//   Op::WEIGHTS    whether op.wgt holds the edges' weights
constexpr int FLY = 8;

template <class Op>
__device__ __forceinline__ int32_t edge_weight(const Op &op, int64_t e) {
  if constexpr (Op::WEIGHTS) return __builtin_nontemporal_load(op.wgt + e);
  else return 0;
}

// One row [e0, e1): tiles of 64 edges first, first + step, ...
template <class Op>
__device__ __forceinline__ typename Op::A walk_row(const Op &op, const int32_t *__restrict__ col, int64_t e0,
                                                   int64_t e1, int first, int step, const u64 *mask, u64 m) {
  const int lane = threadIdx.x & 63;
  const int64_t stride = (int64_t)step * 64;
  typename Op::A acc = op.zero();
  int64_t e = e0 + (int64_t)first * 64;
  int32_t u = e + lane < e1 ? stream_load(col + e + lane) : -1;
  int32_t w = u >= 0 ? edge_weight(op, e + lane) : 0;
  while (e < e1) {
    const u64 mu = u >= 0 ? mask[u] & m : 0ull;
    const int32_t uc = u, wc = w;
    e += stride;  // the next tile's ids
    u = e + lane < e1 ? stream_load(col + e + lane) : -1;
    w = u >= 0 ? edge_weight(op, e + lane) : 0;
    for (u64 todo = __ballot(mu != 0ull); todo;) {
      typename Op::X x[FLY];
      int32_t ws[FLY];
      bool has[FLY];
#pragma unroll
      for (int k = 0; k < FLY; ++k) {
        has[k] = todo != 0;
        if (todo) {
          const int src = __ffsll((long long)todo) - 1;
          todo &= todo - 1;
          ws[k] = Op::WEIGHTS ? __builtin_amdgcn_readlane(wc, src) : 0;
          x[k] = op.load(__builtin_amdgcn_readlane(uc, src), lane_mask(mu, src));
        }
      }
#pragma unroll
      for (int k = 0; k < FLY; ++k)
        if (has[k]) op.add(acc, x[k], ws[k]);
    }
  }
  return acc;
}

// A wave's entries, their edges walked as one list.  Edges stay in order, so
// a row is finished when the owner of the next contributing edge is another
// entry; entries no edge contributes to end in op.idle().
template <class Op>
__device__ __forceinline__ void walk_list(const Op &op, const Entries &E, const int32_t *__restrict__ col,
                                          const u64 *mask) {
  const int lane = threadIdx.x & 63;
  const int k = E.k;
  const int32_t v = E.v;
  const u64 m = E.m;
  if (k == 1 || E.long_list()) {
    for (int j = 0; j < k; ++j) {
      const int32_t vj = __builtin_amdgcn_readlane(v, j);
      const u64 mj = lane_mask(m, j);
      const int64_t ej = lane_i64(E.e0, j);
      const typename Op::P pre = op.begin(vj, mj);
      op.end(j, vj, mj, pre, walk_row(op, col, ej, ej + lane_i64(E.d, j), 0, 1, mask, mj));
    }
    return;
  }
  const int32_t len = (int32_t)E.total;
  int cur = -1;
  typename Op::A acc = op.zero();
  typename Op::P pre = typename Op::P();
  u64 open = __ballot(lane < k);
  const auto finish = [&]() {
    op.end(cur, __builtin_amdgcn_readlane(v, cur), lane_mask(m, cur), pre, acc);
    open &= ~(1ull << cur);
  };
  for (int32_t t0 = 0; t0 < len; t0 += 64) {
    const int32_t t = t0 + lane;
    const int own = E.owner(t);
    const int64_t e = __shfl((long long)E.e0, own, 64) + (t - __shfl(E.start, own, 64));
    const u64 mo = (u64)__shfl((long long)m, own, 64);
    int32_t u = -1, w = 0;
    u64 mu = 0;
    if (t < len) {
      u = stream_load(col + e);
      w = edge_weight(op, e);
      mu = mask[u] & mo;
    }
    for (u64 todo = __ballot(mu != 0ull); todo;) {
      typename Op::X x[FLY];
      typename Op::P p[FLY];
      int32_t ws[FLY];
      int o[FLY];
      int prev = cur;
#pragma unroll
      for (int q = 0; q < FLY; ++q) {
        o[q] = -1;
        if (todo) {
          const int src = __ffsll((long long)todo) - 1;
          todo &= todo - 1;
          o[q] = __builtin_amdgcn_readlane(own, src);
          ws[q] = Op::WEIGHTS ? __builtin_amdgcn_readlane(w, src) : 0;
          if (o[q] != prev) p[q] = op.begin(__builtin_amdgcn_readlane(v, o[q]), lane_mask(m, o[q]));
          prev = o[q];
          x[q] = op.load(__builtin_amdgcn_readlane(u, src), lane_mask(mu, src));
        }
      }
#pragma unroll
      for (int q = 0; q < FLY; ++q)
        if (o[q] >= 0) {
          if (o[q] != cur) {
            if (cur >= 0) finish();
            cur = o[q];
            pre = p[q];
            acc = op.zero();
          }
          op.add(acc, x[q], ws[q]);
        }
    }
  }
  if (cur >= 0) finish();
  op.idle(v, m, open);
}

// Entries [p0, p3) of a degree-sorted sequence below the BLOCK bin, by the
// waves of the grid: [p0, p1) (WAVE bin) one to a wave, [p1, p2) (G16) four,
// [p2, p3) sixteen -- the chain of dependent reads (entry, offsets, ids,
// masks, rows) is otherwise paid per short row.  body(i, k): entries
// [i, i + k).
constexpr int G16_ROWS = 4, LOW_ROWS = 16;
struct RowSpans {
  int64_t p0, p1, p2, p3;
  __host__ __device__ int64_t waves() const {
    return (p1 - p0) + (p2 - p1 + G16_ROWS - 1) / G16_ROWS + (p3 - p2 + LOW_ROWS - 1) / LOW_ROWS;
  }
};
template <class Body>
__device__ __forceinline__ void for_row_spans(const RowSpans &R, int64_t wave, int64_t waves, Body body) {
  const int64_t w1 = R.p1 - R.p0, w2 = w1 + (R.p2 - R.p1 + G16_ROWS - 1) / G16_ROWS, w3 = R.waves();
  for (int64_t x = wave; x < w3; x += waves) {
    const int64_t w = lane_i64(x, 0);  // wave-uniform
    int64_t i, end;
    int k;
    if (w < w1) {
      i = R.p0 + w;
      k = 1;
      end = R.p1;
    } else if (w < w2) {
      i = R.p1 + (w - w1) * G16_ROWS;
      k = G16_ROWS;
      end = R.p2;
    } else {
      i = R.p2 + (w - w2) * LOW_ROWS;
      k = LOW_ROWS;
      end = R.p3;
    }
    if (i + k > end) k = (int)(end - i);
    body(i, k);
  }
}

// OR of the frontier masks of in-neighbours [b, a1) in tiles of 256 edges,
// every `step`-th edge position a tile's first, until all of w is found; the
// edges looked at are added to `checked` (wave-uniform).
__device__ __forceinline__ u64 pull_tiles(const int32_t *__restrict__ icol, const u64 *__restrict__ front, int64_t b,
                                          int64_t a1, int64_t step, u64 w, u64 &checked) {
  const int lane = threadIdx.x & 63;
  u64 got = 0;
  for (; b < a1 && (w & ~got); b += step) {
    checked += (u64)(a1 - b < 256 ? a1 - b : 256);
    u64 x[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t i = b + k * 64 + lane;
      x[k] = i < a1 ? front[icol[i]] : 0ull;
    }
    u64 y = ((x[0] | x[1]) | (x[2] | x[3])) & w;
    if (__ballot(y != 0ull)) {
      for (int o = 32; o > 0; o >>= 1) y |= __shfl_xor(y, o, 64);
      got |= y;
    }
  }
  return got;
}

// The slots of `want` (per lane: vertex v, 0 where the lane has none) found
// on v's in-neighbours: the first four from the head array, sixteen more
// from the row, then the rows still open by the whole wave.  Rows are sorted
// by decreasing degree, so the hubs that most slots have just reached come
// first and most rows close within the head.  The edges looked at are added
// to `checked` (wave-uniform; all lanes active).
template <typename OffT>
__device__ __forceinline__ u64 pull_vertices(const OffT *__restrict__ ioff, const int32_t *__restrict__ icol,
                                             const int4 *__restrict__ head, const u64 *__restrict__ front, int64_t v,
                                             u64 want, u64 &checked) {
  u64 acc = 0;
  int64_t e = 0, e1 = 0;
  uint32_t seen = 0;
  if (want) {
    const int4 h = head[v];
    const int32_t hu[4] = {h.x, h.y, h.z, h.w};
    u64 x[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = hu[k] >= 0 ? front[hu[k]] : 0ull;
    acc = (x[0] | x[1]) | (x[2] | x[3]);
    // (ids of a short row end in -1)
    seen = 4u - ((uint32_t)h.x >> 31) - ((uint32_t)h.y >> 31) - ((uint32_t)h.z >> 31) - ((uint32_t)h.w >> 31);
    if ((want & ~acc) && h.w >= 0) {
      e = (int64_t)ioff[v] + 4;
      e1 = (int64_t)ioff[v + 1];
      for (int r = 0; r < 4 && e < e1 && (want & ~acc); ++r, e += 4) {
#pragma unroll
        for (int k = 0; k < 4; ++k) x[k] = front[icol[e + k < e1 ? e + k : e1 - 1]];
        acc |= (x[0] | x[1]) | (x[2] | x[3]);
      }
      seen = (uint32_t)(min(e, e1) - (int64_t)ioff[v]);
    }
  }
  checked += (u64)wave_total(seen);
  for (u64 todo = __ballot(e < e1 && (want & ~acc) != 0ull); todo; todo &= todo - 1) {
    const int src = __ffsll((long long)todo) - 1;
    const u64 got = pull_tiles(icol, front, lane_i64(e, src), lane_i64(e1, src), 256, lane_mask(want & ~acc, src), checked);
    if ((int)(threadIdx.x & 63) == src) acc |= got;
  }
  return acc & want;
}

}  // namespace tgk
