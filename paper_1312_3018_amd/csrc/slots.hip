// Multi-source supersteps: up to 64 independent BFS or SSSP queries ("slots")
// advance together over one GPU partition.  Each vertex carries one bit per
// slot (BFS: visited / frontier / next masks) or one distance per slot (SSSP),
// so a frontier vertex's edges are streamed once per superstep for every slot
// that has it on its frontier, instead of once per query.
//
// Slots are independent: a slot joins at any superstep boundary (its root
// enters the next frontier with level 0 at that superstep) and retires once
// its frontier is empty, which is what lets a server admit queries while
// others are running (continuous batching).  A superstep is:
//   expand(Q_t) -> clear(Q_t) -> compact(touched) = Q_{t+1} -> finalize(Q_{t+1})
// where "touched" marks vertices that received any slot bit this superstep.
// A superstep in which every slot is pulled is dense instead: one pass over
// all vertices reads the frontier's masks, writes the next ones into a second
// array and settles them, with no queue; a later push makes the queue from
// the masks.
//
// BFS expands by push and pull (ms.hip).  SSSP pushes small frontiers and, on
// a symmetric graph (a vertex's out-edges are its in-edges, with the same
// weights), pulls large ones: a vertex takes the least dist[u] + w over its
// edges from frontier vertices u for all slots at once, with no atomics.  Levels are kept as one byte per
// vertex and slot, a 64-byte row per vertex, and written out in original ids
// when slots retire: a row is read once for all of them and each slot's
// output is one stream of coalesced stores.  (Writing each level to its
// output as it settled made 64 scattered 4-byte stores per vertex: with the
// initial fills, 1.08 of the 2.93 ms of kernels in a 64-root call on a
// uniform graph of 1,000,003 vertices; the one write-out takes 0.11 ms.)  That
// call: 3.18 ms pushing throughout with its buffers made anew each time, 1.28
// ms so.
#include <string.h>

#include <algorithm>

#include "slots.h"

using namespace tgk;

namespace tg {
namespace {

inline unsigned nblk(int64_t n) { return (unsigned)std::max<int64_t>((n + BLOCK - 1) / BLOCK, 1); }

__device__ __forceinline__ void touch(uint32_t *touched, int32_t v) {
  const uint32_t bit = 1u << (v & 31);
  if (!(touched[v >> 5] & bit)) atomicOr(touched + (v >> 5), bit);
}

// Relax every slot on v's frontier mask over v's edges; a lowered distance
// puts the slot on the neighbour's next mask.
//
// An edge whose frontier vertex has several slots takes a wave step with
// lane = slot: the neighbour's 256-byte distance row is read and lowered with
// coalesced accesses, eight edges in flight.  With fewer than ROW_SLOTS slots
// a lane takes the edge by itself and walks them.  Edges come as lists of a
// wave's queue entries (low degrees) or as 64-edge tiles of a long row's
// chunk.  The atomic minimum returns nothing: a lane whose candidate beats
// the distance it read marks the slot, whether or not its own minimum won --
// either way that distance dropped in this superstep.
// RMAT-18, 64 roots: 11.0 ms of launches per call with a lane per edge
// throughout, 7.0 ms so, 2.9 ms with large frontiers pulled.
constexpr int ROW_SLOTS = 4;
constexpr int ROWS_FLY = 8;

struct SsspArgs {
  int32_t *dist;
  u64 *next;
  uint32_t *touched;
  u64 *ovf, *ovf_slots;
};

// Up to 64 edges, one per lane (valid lanes only): neighbour, weight, the
// frontier vertex and its mask.
__device__ __forceinline__ void relax_tile(const SsspArgs &A, bool valid, int32_t nb, int32_t w, int32_t v, u64 m) {
  const int lane = threadIdx.x & 63;
  u64 gained = 0;
  const bool row = valid && __popcll(m) >= ROW_SLOTS;
  int32_t last_v = -1, dv = 0;
  for (u64 todo = __ballot(row); todo;) {
    int32_t cur[ROWS_FLY], from[ROWS_FLY], nbs[ROWS_FLY], ws[ROWS_FLY];
    u64 ms[ROWS_FLY];
    int at[ROWS_FLY];
#pragma unroll
    for (int q = 0; q < ROWS_FLY; ++q) {
      at[q] = -1;
      if (todo) {
        const int src = __ffsll((long long)todo) - 1;
        todo &= todo - 1;
        at[q] = src;
        ms[q] = lane_mask(m, src);
        nbs[q] = __builtin_amdgcn_readlane(nb, src);
        ws[q] = __builtin_amdgcn_readlane(w, src);
        const int32_t vs = __builtin_amdgcn_readlane(v, src);
        if (vs != last_v) {
          dv = A.dist[(int64_t)vs * kSlots + lane];
          last_v = vs;
        }
        from[q] = dv;
        cur[q] = (ms[q] >> lane) & 1ull ? A.dist[(int64_t)nbs[q] * kSlots + lane] : 0;
      }
    }
#pragma unroll
    for (int q = 0; q < ROWS_FLY; ++q)
      if (at[q] >= 0) {
        const bool mine = (ms[q] >> lane) & 1ull;
        // below 2^32: both are below 2^31
        const uint32_t nd = (uint32_t)from[q] + (uint32_t)ws[q];
        const bool fits = nd < (uint32_t)TG_INF;
        const bool better = mine && fits && (int32_t)nd < cur[q];
        if (better) atomicMin(A.dist + (int64_t)nbs[q] * kSlots + lane, (int32_t)nd);
        const u64 g = __ballot(better);
        if (lane == at[q]) gained |= g;
        // a candidate that does not fit marks (vertex, slot); the slot's
        // verdict is taken when it retires (k_ms_ovf_check)
        const u64 o = __ballot(mine && !fits && cur[q] == TG_INF);
        if (o && lane == 0) {
          atomicOr(A.ovf + nbs[q], o);
          atomicOr(A.ovf_slots, o);
        }
      }
  }
  if (valid && !row) {
    const int32_t *dr = A.dist + (int64_t)v * kSlots;
    int32_t *dn = A.dist + (int64_t)nb * kSlots;
    for (u64 bits = m; bits; bits &= bits - 1) {
      const int s = __ffsll((long long)bits) - 1;
      const uint32_t nd = (uint32_t)dr[s] + (uint32_t)w;
      const int32_t c = dn[s];
      if (nd >= (uint32_t)TG_INF) {
        if (c == TG_INF) {
          atomicOr(A.ovf + nb, 1ull << s);
          atomicOr(A.ovf_slots, 1ull << s);
        }
      } else if ((int32_t)nd < c) {
        atomicMin(dn + s, (int32_t)nd);
        gained |= 1ull << s;
      }
    }
  }
  if (gained) {
    if (gained & ~A.next[nb]) atomicOr(A.next + nb, gained);
    touch(A.touched, nb);
  }
}

constexpr int LIST_ROWS = 16;  // queue entries a wave takes below the WAVE bin

__global__ __launch_bounds__(BLOCK) void k_ms_sssp_expand(const Plan *__restrict__ Pp, const int32_t *__restrict__ queue,
                                                          const int64_t *__restrict__ hubpref,
                                                          const int64_t *__restrict__ off,
                                                          const int32_t *__restrict__ col,
                                                          const int32_t *__restrict__ wgt, const u64 *frontier,
                                                          SsspArgs A, int64_t hub_chunk) {
  const Plan &P = load_plan(Pp);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const auto edges = [&](int32_t v, u64 m, int64_t e0, int64_t e1, int64_t stride) {
    for (int64_t e = e0; e < e1; e += stride) {
      const bool ok = e + lane < e1;
      relax_tile(A, ok, ok ? stream_load(col + e + lane) : 0, ok ? stream_load(wgt + e + lane) : 0, v, m);
    }
  };
  // hub chunks, the BLOCK and the WAVE bins: a row's tiles shared by the
  // waves of a block (HUB, BLOCK) or one row to a wave
  const int64_t rows_end = P.vb[BIN_G16];
  // below: LIST_ROWS queue entries to a wave, four waves to a block
  const int64_t q0 = P.pos[BIN_G16], q1 = P.pos[BIN_ZERO];
  const int64_t lists = (q1 - q0 + LIST_ROWS - 1) / LIST_ROWS;
  const int64_t total = rows_end + (lists + 3) / 4;
  for (int64_t vb = blockIdx.x; vb < total; vb += gridDim.x) {
    if (vb < rows_end) {
      const Assign a = assign_work(vb, P, queue, nullptr, hubpref, off, hub_chunk);
      const bool wave_row = a.bin == BIN_WAVE;
      if (!a.ok) continue;  // wave-uniform
      const u64 m = lane_mask(frontier[a.v], 0);
      if (m == 0) continue;
      if (wave_row) edges(a.v, m, a.e_begin, a.e_end, 64);
      else edges(a.v, m, a.e_begin + wv * 64, a.e_end, BLOCK);
      continue;
    }
    const int64_t li = lane_i64((vb - rows_end) * 4 + wv, 0);
    if (li >= lists) continue;
    const int64_t i0 = q0 + li * LIST_ROWS;
    Entries E;
    E.load([&](int64_t i) { return queue[i]; }, [&](int64_t, int32_t v) { return frontier[v]; }, i0,
           (int)(q1 - i0 < LIST_ROWS ? q1 - i0 : LIST_ROWS), off);
    // (rows of the bins here are short: the list fits 32 bits)
    for (int32_t t0 = 0; t0 < (int32_t)E.total; t0 += 64) {
      const int32_t t = t0 + lane;
      const int own = E.owner(t);
      const int64_t e = __shfl((long long)E.e0, own, 64) + (t - __shfl(E.start, own, 64));
      const int32_t v = __shfl(E.v, own, 64);
      const u64 m = (u64)__shfl((long long)E.m, own, 64);
      const bool ok = t < (int32_t)E.total;
      relax_tile(A, ok, ok ? stream_load(col + e) : 0, ok ? stream_load(wgt + e) : 0, v, m);
    }
  }
}

// The same for few slots: lanes by degree bin, a lane walks an edge's slots.
// (Rows that leave most of a wave's lanes without a slot cost more than they
// save, and so do the marks of minima that did not win: those return here.)
__global__ __launch_bounds__(BLOCK) void k_ms_sssp_expand_few(const Plan *__restrict__ Pp,
                                                              const int32_t *__restrict__ queue,
                                                              const int64_t *__restrict__ hubpref,
                                                              const int64_t *__restrict__ off,
                                                              const int32_t *__restrict__ col,
                                                              const int32_t *__restrict__ wgt, const u64 *frontier,
                                                              SsspArgs A, int64_t hub_chunk) {
  const Plan &P = load_plan(Pp);
  const int64_t total = P.vb[NBIN];
  for (int64_t vb = blockIdx.x; vb < total; vb += gridDim.x) {
    const Assign a = assign_work(vb, P, queue, nullptr, hubpref, off, hub_chunk);
    if (!a.ok) continue;
    const u64 m = frontier[a.v];
    if (m == 0) continue;
    const int32_t *dv = A.dist + (int64_t)a.v * kSlots;
    for (int64_t e = a.e_begin + a.lane; e < a.e_end; e += a.stride) {
      const int32_t nb = stream_load(col + e);
      const int32_t w = stream_load(wgt + e);
      int32_t *dn = A.dist + (int64_t)nb * kSlots;
      u64 gained = 0;
      for (u64 bits = m; bits; bits &= bits - 1) {
        const int s = __ffsll((long long)bits) - 1;
        const int64_t nd = (int64_t)dv[s] + (int64_t)w;
        if (nd >= (int64_t)TG_INF) {
          if (dn[s] == TG_INF) {
            atomicOr(A.ovf + nb, 1ull << s);
            atomicOr(A.ovf_slots, 1ull << s);
          }
        } else if (nd < (int64_t)dn[s] && nd < (int64_t)atomicMin(dn + s, (int32_t)nd)) {
          gained |= 1ull << s;
        }
      }
      if (gained && atomicOr(A.next + nb, gained) == 0) atomicOr(A.touched + (nb >> 5), 1u << (nb & 31));
    }
  }
}

__global__ __launch_bounds__(BLOCK) void k_ms_clear(const Plan *__restrict__ Pp, const int32_t *__restrict__ queue,
                                                    u64 *frontier) {
  const int32_t count = Pp->count;
  for (int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x; i < count; i += (int64_t)gridDim.x * BLOCK)
    frontier[queue[i]] = 0;
}

// Levels of the current superstep per slot, one byte each.
struct LevelRow {
  u64 b[kSlots / 8];
};
struct LevelRowWide {
  int32_t v[kSlots];
};

// Bit k of the low byte of x -> byte k of the result all ones.
__device__ __forceinline__ u64 bytes_of_bits(uint32_t x) {
  u64 y = (u64)x * 0x0101010101010101ull & 0x8040201008040201ull;
  y |= y >> 1;
  y |= y >> 2;
  y |= y >> 4;
  return (y & 0x0101010101010101ull) * 255ull;
}

// Note the level of the new bits nb of vertex v.
template <bool WIDE>
__device__ __forceinline__ void put_levels(int64_t v, u64 nb, u64 *__restrict__ lev, int32_t *__restrict__ wide,
                                           const LevelRow &lr, const LevelRowWide &lw) {
  if (WIDE) {
    for (u64 bits = nb; bits; bits &= bits - 1) {
      const int s = __ffsll((long long)bits) - 1;
      wide[v * kSlots + s] = lw.v[s];
    }
  } else {
    u64 *row = lev + v * (kSlots / 8);
#pragma unroll
    for (int k = 0; k < kSlots / 8; ++k) {
      const uint32_t x = (uint32_t)(nb >> (8 * k)) & 255u;
      if (x) {
        const u64 take = bytes_of_bits(x);
        row[k] = (row[k] & ~take) | (lr.b[k] & take);
      }
    }
  }
}

// Blocks of the per-slot sums: wide ones, few of them (each ends with an
// atomic per slot).
constexpr int FT = 1024;
constexpr int FGRID = 512;
inline unsigned fgrid(int64_t n) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + FT - 1) / FT, FGRID)); }

// BFS: settle the bits that arrived this superstep.
template <bool WIDE>
__global__ __launch_bounds__(FT) void k_ms_bfs_finalize(const Plan *__restrict__ Pp,
                                                        const int32_t *__restrict__ queue, u64 *visited,
                                                        u64 *frontier, u64 *next, u64 *__restrict__ lev,
                                                        int32_t *__restrict__ wide, LevelRow lr, LevelRowWide lw,
                                                        const int64_t *__restrict__ off, u64 (*mf)[kSlots],
                                                        u64 (*other)[kSlots]) {
  const int32_t count = Pp->count;
  u64 acc = 0;
  for (int64_t b = (int64_t)blockIdx.x * FT; b < count; b += (int64_t)gridDim.x * FT) {
    const int64_t i = b + threadIdx.x;
    u64 nb = 0;
    uint32_t edges = 0;
    if (i < count) {
      const int32_t v = queue[i];
      const u64 seen = visited[v];
      nb = next[v] & ~seen;
      next[v] = 0;
      visited[v] = seen | nb;
      frontier[v] = nb;
      edges = (uint32_t)(off[v + 1] - off[v]) + 1u;
      put_levels<WIDE>(v, nb, lev, wide, lr, lw);
    }
    add_by_slot(nb, edges, acc);
  }
  publish_by_slot<FT>(acc, mf, other);
}

// BFS, dense superstep: pull the slots of `take` for every vertex below
// `rows` (hubs' bits are already in `next`), settle them and write the next
// frontier masks of all n vertices.  With `joins`, `next` may hold the bits
// of slots that join.
template <typename OffT, bool WIDE>
__global__ __launch_bounds__(FT) void k_ms_bfs_dense(const OffT *__restrict__ ioff, const int32_t *__restrict__ icol,
                                                     const int4 *__restrict__ head, const u64 *__restrict__ front,
                                                     u64 *__restrict__ front_new, u64 *__restrict__ visited,
                                                     u64 *__restrict__ next, int joins, u64 *__restrict__ lev,
                                                     int32_t *__restrict__ wide, LevelRow lr, LevelRowWide lw,
                                                     const int64_t *__restrict__ off, u64 take, int64_t hubs,
                                                     int64_t rows, int64_t n, u64 (*mf)[kSlots],
                                                     u64 (*other)[kSlots], unsigned long long *work) {
  u64 acc = 0, checked = 0, examined = 0;
  for (int64_t vb = (int64_t)blockIdx.x * FT; vb < n; vb += (int64_t)gridDim.x * FT) {
    const int64_t v = vb + threadIdx.x;
    const u64 seen = v < n ? visited[v] : 0ull;
    const u64 want = v >= hubs && v < rows ? take & ~seen : 0ull;
    examined += (u64)__popcll(__ballot(want != 0ull));
    u64 nb = pull_vertices(ioff, icol, head, front, v, want, checked);
    uint32_t edges = 0;
    if (v < n) {
      if (joins || v < hubs) {
        const u64 x = next[v];
        if (x) {
          next[v] = 0;
          nb |= x & ~seen;
        }
      }
      front_new[v] = nb;
      if (nb) {
        visited[v] = seen | nb;
        edges = (uint32_t)(off[v + 1] - off[v]) + 1u;
        put_levels<WIDE>(v, nb, lev, wide, lr, lw);
      }
    }
    add_by_slot(nb, edges, acc);
  }
  __shared__ u64 pulls[FT / 64][2];
  if ((threadIdx.x & 63) == 0) {
    pulls[threadIdx.x >> 6][0] = checked;
    pulls[threadIdx.x >> 6][1] = examined;
  }
  publish_by_slot<FT>(acc, mf, other);  // (its barrier orders `pulls` too)
  if (threadIdx.x >= 64 && threadIdx.x < 66) {
    u64 x = 0;
    for (int k = 0; k < FT / 64; ++k) x += pulls[k][threadIdx.x - 64];
    if (x) stat_add(stat_counter(work, threadIdx.x == 64 ? MS_CHECKED : MS_EXAMINED), x);
  }
}

// From masks to the bitmap a queue is compacted from.
__global__ __launch_bounds__(BLOCK) void k_ms_touch(const u64 *__restrict__ front, int64_t n, uint32_t *touched) {
  const int lane = threadIdx.x & 63;
  const int64_t v = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  const u64 m = __ballot(v < n && front[v] != 0ull);
  if (lane == 0 && (uint32_t)m) touched[v >> 5] = (uint32_t)m;
  if (lane == 32 && (uint32_t)(m >> 32)) touched[v >> 5] = (uint32_t)(m >> 32);
}

// From one byte per level to int32 (a slot is about to pass level 254).
__global__ __launch_bounds__(BLOCK) void k_ms_widen(const uint8_t *__restrict__ lev, int64_t count,
                                                    int32_t *__restrict__ wide) {
  for (int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x; i < count; i += (int64_t)gridDim.x * BLOCK)
    wide[i] = lev[i];
}

// An SSSP frontier, per thread or (the block's part) published: the OR of its
// masks, its edges, its (vertex, slot) pairs and their edges (see MsState and
// MS_PAIRS; the latter on 64 lines, as thousands of blocks add to them).  (Sums
// of 32 bits where they fit: a pulled superstep takes 205 us so, as without
// the last two, 213 with all in 64 bits.)
struct FrontierSums {
  u64 any, edges, relax;
  uint32_t pairs;
  template <class T>
  __device__ __forceinline__ void add(u64 mask, T deg) {
    any |= mask;
    edges += deg;
    const uint32_t k = deg ? (uint32_t)__popcll(mask) : 0u;
    pairs += k;
    relax += (u64)k * deg;
  }
};
template <int THREADS>
__device__ __forceinline__ void publish_frontier(FrontierSums F, u64 (*mf)[kSlots], u64 (*other)[kSlots],
                                                 unsigned long long *work) {
  __shared__ FrontierSums red[THREADS / 64];
  for (int o = 32; o > 0; o >>= 1) {
    F.any |= __shfl_xor(F.any, o, 64);
    F.edges += __shfl_xor(F.edges, o, 64);
    F.pairs += __shfl_xor(F.pairs, o, 64);
    F.relax += __shfl_xor(F.relax, o, 64);
  }
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = F;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < THREADS / 64; ++k) {
      F.any |= red[k].any;
      F.edges += red[k].edges;
      F.pairs += red[k].pairs;
      F.relax += red[k].relax;
    }
    u64 *mine = mf[blockIdx.x % MF_COPIES];
    if (F.any & ~__hip_atomic_load(mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicOr(mine, F.any);
    if (F.edges) atomicAdd(mine + 1, F.edges);
    if (F.pairs) stat_add(stat_counter(work, MS_PAIRS), (u64)F.pairs);
    if (F.relax) stat_add(stat_counter(work, MS_EDGES), F.relax);
    if (blockIdx.x == 0)
      for (int c = 0; c < MF_COPIES; ++c) other[c][0] = other[c][1] = 0ull;
  }
}

// SSSP: the next frontier is whatever slot improved; distances stay in place.
__global__ __launch_bounds__(FT) void k_ms_sssp_finalize(const Plan *__restrict__ Pp,
                                                         const int32_t *__restrict__ queue, u64 *frontier, u64 *next,
                                                         const int64_t *__restrict__ off, u64 (*mf)[kSlots],
                                                         u64 (*other)[kSlots], unsigned long long *work) {
  const int32_t count = Pp->count;
  FrontierSums F{0, 0, 0, 0};
  for (int64_t i = (int64_t)blockIdx.x * FT + threadIdx.x; i < count; i += (int64_t)gridDim.x * FT) {
    const int32_t v = queue[i];
    const u64 nb = next[v];
    next[v] = 0;
    frontier[v] = nb;
    F.add(nb, (u64)(off[v + 1] - off[v]));
  }
  publish_frontier<FT>(F, mf, other, work);
}

// SSSP, dense superstep on a symmetric graph: rows are distance rows, a
// row's value the least dist[u] + w over the edges from frontier vertices u.
// Distances are read and written in place: a neighbour lowered meanwhile is
// on the next frontier, so that its new value is pulled then.
struct MinOp {
  using X = int32_t;
  using A = uint32_t;  // ~0: no candidate; at least TG_INF: one that does not fit
  using P = int32_t;
  static constexpr bool WEIGHTS = true;
  const int32_t *wgt;
  int32_t *dist;
  u64 *front_new, *next;
  int joins;
  u64 *ovf, *ovf_slots;
  int32_t deg;  // per lane: the entry's edges
  FrontierSums *sums;

  __device__ __forceinline__ A zero() const { return ~0u; }
  __device__ __forceinline__ P begin(int32_t v, u64) const { return dist[(int64_t)v * kSlots + (threadIdx.x & 63)]; }
  __device__ __forceinline__ X load(int32_t u, u64) const { return dist[(int64_t)u * kSlots + (threadIdx.x & 63)]; }
  // below 2^32: both are below 2^31
  __device__ __forceinline__ void add(A &acc, X x, int32_t w) const {
    acc = min(acc, x == TG_INF ? ~0u : (uint32_t)x + (uint32_t)w);
  }
  // Slots that improve on `own`, and the marks of those that overflow.
  __device__ __forceinline__ u64 gains(int32_t v, P own, A acc, bool &better) const {
    const bool fits = acc < (uint32_t)TG_INF;
    better = fits && (int32_t)acc < own;
    const u64 o = __ballot(!fits && acc != ~0u && own == TG_INF);
    if (o && (threadIdx.x & 63) == 0) {
      atomicOr(ovf + v, o);
      atomicOr(ovf_slots, o);
    }
    return __ballot(better);
  }
  __device__ __forceinline__ void end(int j, int32_t v, u64, P own, A acc) const {
    const int lane = threadIdx.x & 63;
    bool better;
    u64 g = gains(v, own, acc, better);
    if (better) dist[(int64_t)v * kSlots + lane] = (int32_t)acc;
    if (joins) {
      g |= next[v];
      if (lane == 0) next[v] = 0;
    }
    if (lane == 0) {
      front_new[v] = g;
      if (g) sums->add(g, (uint32_t)__builtin_amdgcn_readlane(deg, j));
    }
  }
  __device__ __forceinline__ void idle(int32_t v, u64, u64 open) const {
    const int lane = threadIdx.x & 63;
    if (!((open >> lane) & 1ull)) return;
    u64 g = 0;
    if (joins) {
      g = next[v];
      next[v] = 0;
    }
    front_new[v] = g;
    if (g) sums->add(g, (uint32_t)deg);
  }
};

// The rows of the largest degrees, SSSP_HUB_WAVES waves each; improved slots
// go to `next`.
constexpr int SSSP_HUB_WAVES = 16;
__global__ __launch_bounds__(BLOCK) void k_ms_sssp_pull_hubs(const int64_t *__restrict__ off,
                                                             const int32_t *__restrict__ col, const u64 *front,
                                                             int64_t hubs, MinOp op) {
  const int lane = threadIdx.x & 63;
  const int64_t nw = (int64_t)gridDim.x * (BLOCK / 64);
  for (int64_t t = (int64_t)blockIdx.x * (BLOCK / 64) + (threadIdx.x >> 6); t < hubs * SSSP_HUB_WAVES; t += nw) {
    const int32_t v = (int32_t)lane_i64(t / SSSP_HUB_WAVES, 0);
    const int part = __builtin_amdgcn_readfirstlane((int)(t % SSSP_HUB_WAVES));
    const uint32_t acc = walk_row(op, col, lane_i64(off[v], 0), lane_i64(off[v + 1], 0), part, SSSP_HUB_WAVES, front,
                                  ~0ull);
    bool better;
    const u64 g = op.gains(v, op.begin(v, ~0ull), acc, better);
    if (better) atomicMin(op.dist + (int64_t)v * kSlots + lane, (int32_t)acc);
    if (g && lane == 0) atomicOr(op.next + v, g);
  }
}

__global__ __launch_bounds__(BLOCK) void k_ms_sssp_pull(const int64_t *__restrict__ off,
                                                        const int32_t *__restrict__ col, const u64 *front,
                                                        int64_t hubs, RowSpans R, MinOp op, u64 (*mf)[kSlots],
                                                        u64 (*other)[kSlots], unsigned long long *work) {
  FrontierSums F{0, 0, 0, 0};
  op.sums = &F;
  for (int64_t v = (int64_t)blockIdx.x * BLOCK + threadIdx.x; v < hubs; v += (int64_t)gridDim.x * BLOCK) {
    const u64 g = op.next[v];
    if (g) {
      op.next[v] = 0;
      F.add(g, (u64)(off[v + 1] - off[v]));
    }
    op.front_new[v] = g;
  }
  for_row_spans(R, ((int64_t)blockIdx.x * BLOCK + threadIdx.x) >> 6, ((int64_t)gridDim.x * BLOCK) >> 6,
                [&](int64_t i, int k) {
                  Entries E;
                  E.load([](int64_t x) { return (int32_t)x; }, [](int64_t, int32_t) { return ~0ull; }, i, k, off);
                  op.deg = (int32_t)E.d;
                  walk_list(op, E, col, front);
                });
  publish_frontier<BLOCK>(F, mf, other, work);
}

struct Roots {
  int32_t v[kSlots];
};

// Slots first.. join: their roots get the slot bits on the next frontier.
__global__ __launch_bounds__(kSlots) void k_ms_join(u64 *next, uint32_t *touched, int32_t *dist, Roots roots,
                                                    int first, int count) {
  const int k = threadIdx.x;
  if (k >= count) return;
  const int32_t r = roots.v[k];
  atomicOr(next + r, 1ull << (first + k));
  atomicOr(touched + (r >> 5), 1u << (r & 31));
  if (dist) dist[(int64_t)r * kSlots + first + k] = 0;
}

// Overflow verdict of retiring slots: bit s of *bad is set if some vertex
// received an overflowing candidate from slot s and stayed unreached (its
// true distance is finite but does not fit below INT32_MAX).  A vertex whose
// candidate overflowed but that was reached otherwise has its exact
// distance: path prefixes only grow, so an overflowing prefix never leads to
// a shorter path.
__global__ __launch_bounds__(BLOCK) void k_ms_ovf_check(const u64 *__restrict__ ovf, const int32_t *__restrict__ dist,
                                                        int64_t n, u64 mask, u64 *bad) {
  u64 found = 0;
  for (int64_t v = (int64_t)blockIdx.x * BLOCK + threadIdx.x; v < n; v += (int64_t)gridDim.x * BLOCK) {
    u64 bits = ovf[v] & mask;
    while (bits) {
      const int s = __ffsll((long long)bits) - 1;
      bits &= bits - 1;
      if (dist[v * kSlots + s] == TG_INF) found |= 1ull << s;
    }
  }
  for (int o = 32; o > 0; o >>= 1) found |= __shfl_xor(found, o, 64);
  if ((threadIdx.x & 63) == 0 && found) atomicOr(bad, found);
}

// Retiring slots: drop their bits / reset their distances and overflow
// marks everywhere (distances a row at a time, lane = slot).
// Block 0 of the last launch of a retirement leaves the counters' sums in
// pinned memory: 64 lines each are slow to read from the host.
__device__ __forceinline__ void report_work(const unsigned long long *work, unsigned long long *sums) {
  const int k = threadIdx.x >> 6;
  if (blockIdx.x != 0 || k >= MS_COUNTERS) return;
  const u64 x = wave_sum((u64)work[(size_t)k * STAT_SPAN + (threadIdx.x & 63) * STAT_STRIDE]);
  if ((threadIdx.x & 63) == 0) sums[k] = x;
}
__global__ __launch_bounds__(BLOCK) void k_ms_release(u64 *visited, u64 *ovf, int64_t n, u64 mask,
                                                      const unsigned long long *work, unsigned long long *sums) {
  if (sums) report_work(work, sums);
  for (int64_t v = (int64_t)blockIdx.x * BLOCK + threadIdx.x; v < n; v += (int64_t)gridDim.x * BLOCK) {
    if (visited) visited[v] &= ~mask;
    if (ovf) ovf[v] &= ~mask;
  }
}
// A launch's threads are counted in 32 bits: 64 a vertex would wrap around,
// unreported, from 2^26 vertices on.  The release has a thread per distance up
// to half of that and strides beyond.  (16384 blocks that stride are done
// sooner, one slot 7 instead of 17 us on RMAT-18 and 110 instead of 227 on
// 2^22 vertices, but the server then completes more supersteps of fewer queries
// each: the eight graphs of the serving benchmark, 2,000 queries/s offered,
// 1,245 instead of 1,370 served/s.)
constexpr int64_t ROW_GRID = 16384, RELEASE_GRID = 1 << 23;
__global__ __launch_bounds__(BLOCK) void k_ms_release_dist(int32_t *dist, int64_t n, u64 mask,
                                                           const unsigned long long *work, unsigned long long *sums) {
  report_work(work, sums);
  if (!((mask >> (threadIdx.x & (kSlots - 1))) & 1ull)) return;
  for (int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x; i < n * kSlots; i += (int64_t)gridDim.x * BLOCK)
    dist[i] = TG_INF;
}

// Levels of the slots in `mask` into their outputs, vertices in original id
// order: the 64-byte row is read once, and a slot's stores are coalesced.
__global__ __launch_bounds__(BLOCK) void k_ms_bfs_collect(const u64 *__restrict__ visited,
                                                          const uint4 *__restrict__ lev,
                                                          const int32_t *__restrict__ wide,
                                                          const int32_t *__restrict__ l_of_g, int64_t V, u64 mask,
                                                          SlotTable tab) {
  const int64_t gid = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (gid >= V) return;
  const int32_t l = l_of_g[gid];
  const u64 seen = visited[l];
  if (wide) {
    for (u64 bits = mask; bits; bits &= bits - 1) {
      const int s = __ffsll((long long)bits) - 1;
      tab.out[s][gid] = (seen >> s) & 1ull ? wide[(int64_t)l * kSlots + s] : TG_INF;
    }
    return;
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (!((mask >> (16 * k)) & 0xFFFFull)) continue;
    const uint4 x = lev[(int64_t)l * 4 + k];
    const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int s = 16 * k + q;
      if ((mask >> s) & 1ull)
        __builtin_nontemporal_store((seen >> s) & 1ull ? (int32_t)((w[q >> 2] >> (8 * (q & 3))) & 255u) : TG_INF,
                                    tab.out[s] + gid);
    }
  }
}

// Distances of the slots in `mask` into their outputs: a block takes 64
// vertices in original id order at a time, reads their rows (lane = slot)
// into LDS and writes each slot's 64 values (lane = vertex).
__global__ __launch_bounds__(BLOCK) void k_ms_sssp_collect(const int32_t *__restrict__ dist,
                                                           const int32_t *__restrict__ l_of_g, int64_t V, u64 mask,
                                                           SlotTable tab) {
  __shared__ int32_t tile[64][kSlots + 1];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int64_t g0 = (int64_t)blockIdx.x * 64; g0 < V; g0 += (int64_t)gridDim.x * 64) {
    const int32_t l = g0 + lane < V ? l_of_g[g0 + lane] : 0;  // past the end: any row
    int32_t x[16];
#pragma unroll
    for (int j = 0; j < 16; ++j)
      x[j] = dist[(int64_t)__builtin_amdgcn_readlane(l, w * 16 + j) * kSlots + lane];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 16; ++j) tile[w * 16 + j][lane] = x[j];
    __syncthreads();
    if (g0 + lane < V)
      for (int s = w * 16; s < w * 16 + 16; ++s)
        if ((mask >> s) & 1ull) __builtin_nontemporal_store(tile[lane][s], tab.out[s] + g0 + lane);
  }
}

__global__ void k_clear_bits64(u64 *word, u64 mask) {
  if (threadIdx.x == 0) atomicAnd(word, ~mask);
}

__global__ __launch_bounds__(BLOCK) void k_fill_i32_all(int32_t *p, int64_t n, int32_t v) {
  for (int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLOCK) p[i] = v;
}

}  // namespace

SlotEngine::~SlotEngine() {
  if (h_state) TG_QUIET(hipHostFree(h_state));
  if (h_ovf) TG_QUIET(hipHostFree(h_ovf));
}

int SlotEngine::init(tg_partition *part, int kind_, hipStream_t stream) {
  const GpuPart &g = part->gpu;
  if (kind_ == kSlotSssp && !g.out.w) return set_error(TG_EUNSUPPORTED, "sssp: the graph was loaded without weights");
  const uint64_t gen = ws.gen;
  const bool kept = p == part && kind == kind_ && cap_n == g.n && clean;
  p = part;
  kind = kind_;
  s = stream;
  TG_TRY(ws.ensure(g, 0));
  memset(&tab, 0, sizeof(tab));
  busy = alive = 0;
  step = 0;
  have_queue = dense = joined = false;
  done = SearchWork();
  if (ws.gen != gen) memset(counted, 0, sizeof(counted));  // (new buffers, cleared)
  if (kept) {
    // every slot of the last run retired: the buffers are as after set-up
    if (ws.gen != gen) ws.plan = &state->plan;
    return TG_OK;
  }
  clean = false;
  is_wide = false;
  wide = nullptr;
  arena.release();
  const int64_t n = std::max<int64_t>(g.n, 1);
  TG_TRY(dalloc(arena, &front[0], (size_t)n));
  TG_TRY(dalloc(arena, &front[1], (size_t)n));
  cur = 0;
  TG_TRY(dalloc(arena, &next, (size_t)n));
  TG_TRY(dalloc(arena, &state, 1));
  ws.plan = &state->plan;
  TG_HIP(hipMemset(state, 0, sizeof(MsState)));
  TG_HIP(hipMemset(front[0], 0, (size_t)n * sizeof(u64)));
  TG_HIP(hipMemset(front[1], 0, (size_t)n * sizeof(u64)));
  TG_HIP(hipMemset(next, 0, (size_t)n * sizeof(u64)));
  if (kind == kSlotBfs) {
    TG_TRY(dalloc(arena, &visited, (size_t)n));
    TG_HIP(hipMemset(visited, 0, (size_t)n * sizeof(u64)));
    TG_TRY(dalloc(arena, &lev, (size_t)n * kSlots));
  } else {
    TG_TRY(dalloc(arena, &ovf, (size_t)n));
    TG_TRY(dalloc(arena, &ovf_slots, 2));
    TG_HIP(hipMemset(ovf, 0, (size_t)n * sizeof(u64)));
    TG_HIP(hipMemset(ovf_slots, 0, 2 * sizeof(u64)));
    TG_TRY(dalloc(arena, &dist, (size_t)n * kSlots));
    hipLaunchKernelGGL(k_fill_i32_all, dim3(2048), dim3(BLOCK), 0, s, dist, n * kSlots, TG_INF);
    TG_HIP(hipGetLastError());
  }
  if (!h_state) TG_HIP(hipHostMalloc((void **)&h_state, sizeof(MsState), hipHostMallocDefault));
  if (!h_ovf) TG_HIP(hipHostMalloc((void **)&h_ovf, (2 + MS_COUNTERS) * sizeof(u64), hipHostMallocDefault));
  TG_HIP(hipMemset(ws.bits_a, 0, ws.nwords * sizeof(uint32_t)));
  TG_HIP(hipMemset(ws.counters, 0, 64 * sizeof(uint32_t)));
  TG_HIP(hipMemset(ws.work, 0, (size_t)STAT_COUNTERS * STAT_SPAN * sizeof(unsigned long long)));
  memset(counted, 0, sizeof(counted));
  // the clears above are on the null stream, not ordered before work on a
  // non-blocking stream such as a server lane's
  TG_HIP(hipDeviceSynchronize());
  cap_n = g.n;
  clean = true;
  return TG_OK;
}

int SlotEngine::free_slot() const {
  for (int k = 0; k < kSlots; ++k)
    if (!((busy >> k) & 1ull)) return k;
  return -1;
}

int SlotEngine::join(int first, int count, const int32_t *roots_local) {
  Roots roots;
  for (int k = 0; k < count; ++k) {
    roots.v[k] = roots_local[k];
    // the root settles (level 0) in the next superstep, which first advances
    // the counter if a frontier is in flight
    tab.join[first + k] = (int32_t)(have_queue ? step + 1 : step);
    mu[first + k] = p->gpu.m;
    busy |= 1ull << (first + k);
  }
  clean = false;
  joined = true;
  hipLaunchKernelGGL(k_ms_join, dim3(1), dim3(kSlots), 0, s, next, ws.bits_a, kind == kSlotSssp ? dist : nullptr,
                     roots, first, count);
  TG_HIP(hipGetLastError());
  return TG_OK;
}

int SlotEngine::superstep(u64 *finished) {
  TG_TRY(launch_step());
  return finish_step(finished);
}

int SlotEngine::widen() {
  const int64_t count = std::max<int64_t>(p->gpu.n, 1) * kSlots;
  if (!wide) TG_TRY(dalloc(arena, &wide, (size_t)count));
  hipLaunchKernelGGL(k_ms_widen, dim3(4096), dim3(BLOCK), 0, s, lev, count, wide);
  TG_HIP(hipGetLastError());
  is_wide = true;
  return TG_OK;
}

// Levels of this superstep, per slot.
static void level_rows(const SlotEngine &E, LevelRow &lr, LevelRowWide &lw) {
  memset(&lr, 0, sizeof(lr));
  for (int k = 0; k < kSlots; ++k) {
    lw.v[k] = (int32_t)E.step - E.tab.join[k];
    lr.b[k / 8] |= (u64)(lw.v[k] & 255) << (8 * (k & 7));
  }
}

// Share of the edges above which an SSSP frontier is pulled: a pull reads
// every vertex's row of ids and masks, a push only the frontier's, but with
// atomics.
constexpr u64 SSSP_PULL_SHARE = 8;  // one in
// Up to this many slots are pushed edge by edge and not pulled.  (ms a call,
// edge by edge / rows and pulls: symmetric RMAT-20, 1 slot 1.65 / 3.90, 4 3.29
// / 4.55; RMAT-22, 1 5.37 / 11.3, 4 12.5 / 15.6; uniform of 2^20, 4 4.58 / 5.71;
// directed RMAT-20, 1 1.40 / 2.05, 8 4.14 / 7.60.)
int sssp_few(const GpuPart &g) { return g.in_alias ? 4 : 16; }

int SlotEngine::launch_step() {
  const GpuPart &g = p->gpu;
  u64 pulled = 0, mf[kSlots] = {};
  bool all_pull = false;
  if (have_queue && alive) {
    if (kind == kSlotBfs) {
      for (int c = 0; c < MF_COPIES; ++c)
        for (int k = 0; k < kSlots; ++k) mf[k] += h_state->mf[step & 1][c][k];
      pulled = ms_pull_slots(mf, mu, alive, p->tune);
      all_pull = pulled == alive;
    } else {
      all_pull = g.in_alias && __builtin_popcountll(alive) > sssp_few(g) && pull_edges * SSSP_PULL_SHARE > (u64)g.m;
    }
    // a queue made from the masks would miss the slots that join
    if (dense && joined) all_pull = true;
    if (all_pull) pulled = alive;
    // what this superstep does, for the call's statistics
    if (kind == kSlotBfs) {
      done.steps += pulled ? 1.0 : 0.0;
    } else {
      done.read += (double)(all_pull ? (u64)g.m : pull_edges);
      done.pulls += all_pull ? 1.0 : 0.0;
    }
  }
  if (kind == kSlotBfs && !is_wide) {
    const int64_t next_step = have_queue ? step + 1 : step;
    for (int k = 0; k < kSlots; ++k)
      if (((busy >> k) & 1ull) && (int32_t)next_step - tab.join[k] > 254) {
        TG_TRY(widen());
        break;
      }
  }
  TG_TRY(all_pull ? launch_dense() : launch_sparse(pulled));
  joined = false;
  TG_HIP(hipMemcpyAsync(h_state, state, sizeof(MsState), hipMemcpyDeviceToHost, s));
  return TG_OK;
}

// One pass over all vertices, every slot pulled.
int SlotEngine::launch_dense() {
  const GpuPart &g = p->gpu;
  const u64 *now = front[cur];
  u64 *then = front[cur ^ 1];
  ++step;
  u64(*mf)[kSlots] = state->mf[step & 1], (*other)[kSlots] = state->mf[(step + 1) & 1];
  const int64_t hubs = hub_rows(g);
  const int joins = joined ? 1 : 0;
  if (joined) TG_HIP(hipMemsetAsync(ws.bits_a, 0, ws.nwords * sizeof(uint32_t), s));  // the joins' marks
  const int tk = ktimer_start(s);
  if (kind == kSlotBfs) {
    TG_TRY(ms_pull_hubs(g, ws, nullptr, now, visited, next, alive, s));
    LevelRow lr;
    LevelRowWide lw;
    level_rows(*this, lr, lw);
    const int64_t rows = g.in_alias ? g.out_bins.bstart[BIN_ZERO] : g.n;
    const int4 *head = reinterpret_cast<const int4 *>(g.in_head);
    const dim3 grid(fgrid(g.n)), block(FT);
    u64 *l8 = reinterpret_cast<u64 *>(lev);
    if (g.in_off32 && !is_wide)
      hipLaunchKernelGGL((k_ms_bfs_dense<int32_t, false>), grid, block, 0, s, g.in_off32, g.in.col, head, now, then,
                         visited, next, joins, l8, wide, lr, lw, g.out.off, alive, hubs, rows, g.n, mf, other, ws.work);
    else if (g.in_off32)
      hipLaunchKernelGGL((k_ms_bfs_dense<int32_t, true>), grid, block, 0, s, g.in_off32, g.in.col, head, now, then,
                         visited, next, joins, l8, wide, lr, lw, g.out.off, alive, hubs, rows, g.n, mf, other, ws.work);
    else if (!is_wide)
      hipLaunchKernelGGL((k_ms_bfs_dense<int64_t, false>), grid, block, 0, s, g.in.off, g.in.col, head, now, then,
                         visited, next, joins, l8, wide, lr, lw, g.out.off, alive, hubs, rows, g.n, mf, other, ws.work);
    else
      hipLaunchKernelGGL((k_ms_bfs_dense<int64_t, true>), grid, block, 0, s, g.in.off, g.in.col, head, now, then,
                         visited, next, joins, l8, wide, lr, lw, g.out.off, alive, hubs, rows, g.n, mf, other, ws.work);
  } else {
    MinOp op{g.out.w, dist, then, next, joins, ovf, ovf_slots, 0, nullptr};
    if (hubs > 0)
      hipLaunchKernelGGL(k_ms_sssp_pull_hubs, dim3((unsigned)std::min<int64_t>(hubs * SSSP_HUB_WAVES / 4, 16384)),
                         dim3(BLOCK), 0, s, g.out.off, g.out.col, now, hubs, op);
    const RowSpans R{hubs, g.out_bins.bstart[BIN_G16], g.out_bins.bstart[BIN_G4], g.n};
    hipLaunchKernelGGL(k_ms_sssp_pull, dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>((R.waves() + 3) / 4, 8192))),
                       dim3(BLOCK), 0, s, g.out.off, g.out.col, now, hubs, R, op, mf, other, ws.work);
  }
  ktimer_stop(tk, s, kind == kSlotBfs ? "msbfs_expand" : "mssssp_expand");
  TG_HIP(hipGetLastError());
  cur ^= 1;
  dense = true;
  return TG_OK;
}

// Over the frontier's queue, slots of `pulled` pulled and the others pushed.
int SlotEngine::launch_sparse(u64 pulled) {
  const GpuPart &g = p->gpu;
  const Tuning &t = p->tune;
  Plan hp = h_state->plan;
  u64 *frontier = front[cur];
  if (have_queue && dense && alive) {
    // the queue of the frontier, from its masks; its size stays on the device
    hipLaunchKernelGGL(k_ms_touch, dim3(nblk(g.n)), dim3(BLOCK), 0, s, frontier, g.n, ws.bits_a);
    TG_TRY(frontier_compact(g, ws, 1, ws.bits_a, nullptr, ws.queue, nullptr, 0, s));
    TG_TRY(frontier_plan(g, ws, ws.queue, t, s, false));
    hp.count = (int32_t)std::min<int64_t>(g.n, 1 << 18);
    for (int b = 1; b <= NBIN; ++b) hp.vb[b] = 4096;
  }
  if (have_queue && hp.count > 0 && (alive || !dense)) {
    const int tk = ktimer_start(s);
    if (kind == kSlotBfs) {
      TG_TRY(ms_expand(g, ws, t, hp, ws.queue, frontier, visited, next, alive, pulled, s));
    } else if (hp.vb[NBIN] > 0 && __builtin_popcountll(alive) <= sssp_few(g)) {
      hipLaunchKernelGGL(k_ms_sssp_expand_few, dim3(launch_grid(hp.vb[NBIN])), dim3(BLOCK), 0, s, ws.plan, ws.queue,
                         ws.hubpref, g.out.off, g.out.col, g.out.w, frontier,
                         SsspArgs{dist, next, ws.bits_a, ovf, ovf_slots}, t.hub_chunk);
    } else if (hp.vb[NBIN] > 0) {
      const int64_t lists = (hp.pos[BIN_ZERO] - hp.pos[BIN_G16] + LIST_ROWS - 1) / LIST_ROWS;
      hipLaunchKernelGGL(k_ms_sssp_expand, dim3(launch_grid(hp.vb[BIN_G16] + (lists + 3) / 4)), dim3(BLOCK), 0, s,
                         ws.plan, ws.queue, ws.hubpref, g.out.off, g.out.col, g.out.w, frontier,
                         SsspArgs{dist, next, ws.bits_a, ovf, ovf_slots}, t.hub_chunk);
    }
    ktimer_stop(tk, s, kind == kSlotBfs ? "msbfs_expand" : "mssssp_expand");
    hipLaunchKernelGGL(k_ms_clear, dim3(nblk(std::min<int64_t>(hp.count, 1 << 20))), dim3(BLOCK), 0, s, ws.plan,
                       ws.queue, frontier);
    TG_HIP(hipGetLastError());
  }
  if (have_queue) ++step;
  dense = false;
  // next frontier: every vertex that received a slot bit (mode 1 takes and clears)
  TG_TRY(frontier_compact(g, ws, 1, ws.bits_a, nullptr, ws.queue, nullptr, 0, s));
  TG_TRY(frontier_plan(g, ws, ws.queue, t, s, false));
  u64(*mf)[kSlots] = state->mf[step & 1], (*other)[kSlots] = state->mf[(step + 1) & 1];
  if (kind == kSlotBfs) {
    LevelRow lr;
    LevelRowWide lw;
    level_rows(*this, lr, lw);
    u64 *l8 = reinterpret_cast<u64 *>(lev);
    if (is_wide)
      hipLaunchKernelGGL(k_ms_bfs_finalize<true>, dim3(fgrid(g.n)), dim3(FT), 0, s, ws.plan, ws.queue, visited,
                         frontier, next, l8, wide, lr, lw, g.out.off, mf, other);
    else
      hipLaunchKernelGGL(k_ms_bfs_finalize<false>, dim3(fgrid(g.n)), dim3(FT), 0, s, ws.plan, ws.queue, visited,
                         frontier, next, l8, wide, lr, lw, g.out.off, mf, other);
  } else {
    hipLaunchKernelGGL(k_ms_sssp_finalize, dim3(fgrid(g.n)), dim3(FT), 0, s, ws.plan, ws.queue, frontier, next,
                       g.out.off, mf, other, ws.work);
  }
  TG_HIP(hipGetLastError());
  return TG_OK;
}

int SlotEngine::finish_step(u64 *finished) {
  TG_HIP(hipStreamSynchronize(s));
  ktimer_flush();
  have_queue = true;
  ++supersteps;
  // a busy slot with no bit on the new frontier has finished
  alive = 0;
  pull_edges = 0;
  for (int c = 0; c < MF_COPIES; ++c) {
    const u64 *mf = h_state->mf[step & 1][c];
    if (kind == kSlotBfs) {
      for (int k = 0; k < kSlots; ++k) {
        if (mf[k]) alive |= 1ull << k;
        mu[k] -= (int64_t)mf[k];
      }
    } else {
      alive |= mf[0];
      pull_edges += mf[1];
    }
  }
  *finished = busy & ~alive;
  return TG_OK;
}

int SlotEngine::retire(u64 mask, u64 *overflow) {
  const GpuPart &g = p->gpu;
  if (overflow) *overflow = 0;
  if (!mask) return TG_OK;
  const unsigned grid = nblk(std::min<int64_t>(g.n, 1 << 20));
  const int64_t V = g.n_global;
  u64 outs = 0;  // retiring slots with an output
  for (int k = 0; k < kSlots; ++k)
    if (((mask >> k) & 1ull) && tab.out[k]) outs |= 1ull << k;
  if (kind == kSlotSssp) {
    if (outs)
      hipLaunchKernelGGL(k_ms_sssp_collect, dim3((unsigned)std::min<int64_t>((V + 63) / 64, ROW_GRID)), dim3(BLOCK), 0,
                         s, dist, g.l_of_g, V, outs, tab);
    // slots that saw an overflowing candidate get the exact verdict
    TG_HIP(hipMemcpyAsync(h_ovf, ovf_slots, sizeof(u64), hipMemcpyDeviceToHost, s));
    TG_HIP(hipStreamSynchronize(s));
    const u64 flagged = h_ovf[0] & mask;
    if (flagged) {
      TG_HIP(hipMemsetAsync(ovf_slots + 1, 0, sizeof(u64), s));
      hipLaunchKernelGGL(k_ms_ovf_check, dim3(grid), dim3(BLOCK), 0, s, ovf, dist, g.n, flagged, ovf_slots + 1);
      hipLaunchKernelGGL(k_clear_bits64, dim3(1), dim3(64), 0, s, ovf_slots, flagged);
      hipLaunchKernelGGL(k_ms_release, dim3(grid), dim3(BLOCK), 0, s, nullptr, ovf, g.n, mask,
                         nullptr, nullptr);
      TG_HIP(hipMemcpyAsync(h_ovf + 1, ovf_slots + 1, sizeof(u64), hipMemcpyDeviceToHost, s));
    }
    hipLaunchKernelGGL(k_ms_release_dist, dim3((unsigned)std::min<int64_t>(nblk(g.n * kSlots), RELEASE_GRID)),
                       dim3(BLOCK), 0, s, dist, g.n, mask, ws.work, h_ovf + 2);
    TG_HIP(hipGetLastError());
    TG_HIP(hipStreamSynchronize(s));
    if (flagged && overflow) *overflow = h_ovf[1] & flagged;
  } else {
    if (outs)
      hipLaunchKernelGGL(k_ms_bfs_collect, dim3(nblk(V)), dim3(BLOCK), 0, s, visited,
                         reinterpret_cast<const uint4 *>(lev), is_wide ? wide : nullptr, g.l_of_g, V, outs, tab);
    hipLaunchKernelGGL(k_ms_release, dim3(grid), dim3(BLOCK), 0, s, visited, nullptr, g.n, mask, ws.work,
                       h_ovf + 2);
    TG_HIP(hipGetLastError());
    TG_HIP(hipStreamSynchronize(s));
  }
  busy &= ~mask;
  for (int k = 0; k < kSlots; ++k)
    if ((mask >> k) & 1ull) tab.out[k] = nullptr;
  if (!busy) {
    is_wide = false;
    clean = true;
  }
  return TG_OK;
}

void slots_drop(tg_partition *p, int kind) {
  delete p->slots[kind];
  p->slots[kind] = nullptr;
}

// Batched BFS / SSSP from a fixed list of roots: chunks of 64 slots that all
// join at superstep 0 and retire together.
int slots_run_batch(tg_partition *p, int kind, const int32_t *roots, int32_t nr, int32_t *out, hipStream_t s,
                    int64_t *supersteps_out, SearchWork *work) {
  if (!p->slots[kind]) {
    p->slots[kind] = new (std::nothrow) SlotEngine();
    if (!p->slots[kind]) return set_error(TG_ENOMEM, "slot engine: out of host memory");
  }
  SlotEngine &E = *p->slots[kind];
  TG_TRY(E.init(p, kind, s));
  const int64_t V = p->g->n;
  int64_t total = 0;
  for (int32_t c0 = 0; c0 < nr; c0 += kSlots) {
    const int32_t cn = std::min<int32_t>(kSlots, nr - c0);
    int32_t local[kSlots];
    for (int32_t k = 0; k < cn; ++k) {
      local[k] = p->h_l_of_g[roots[c0 + k]];
      E.tab.out[k] = out + (int64_t)(c0 + k) * V;
    }
    TG_TRY(E.join(0, cn, local));
    const u64 all = E.busy;
    u64 fin = 0;
    for (int64_t it = 0; fin != all; ++it) {
      if (it > p->gpu.n + 2) return set_error(TG_EDEVICE, "batched run: no convergence");
      TG_TRY(E.superstep(&fin));
    }
    u64 ovf = 0;
    TG_TRY(E.retire(fin, &ovf));
    double now[MS_COUNTERS];
    for (int k = 0; k < MS_COUNTERS; ++k) {
      now[k] = (double)(E.h_ovf[2 + k] - E.counted[k]);
      E.counted[k] = E.h_ovf[2 + k];
    }
    E.done.vertices += now[MS_PAIRS];
    E.done.edges += now[MS_EDGES];
    E.done.checked += now[MS_CHECKED];
    E.done.examined += now[MS_EXAMINED];
    total += E.step;
    E.step = 0;
    E.have_queue = E.dense = false;
    if (ovf) {
      const int k = __builtin_ctzll(ovf);
      return set_error(TG_ERANGE, "sssp_batched: the distances from root %d do not fit below INT32_MAX",
                       roots[c0 + k]);
    }
  }
  if (supersteps_out) *supersteps_out = total;
  E.done.lanes = std::min<int>(nr, kSlots);
  *work = E.done;
  return TG_OK;
}

}  // namespace tg
