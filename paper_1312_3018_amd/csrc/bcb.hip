// Batched Brandes betweenness (section 7.2, Figure 18) for up to 64 sources
// per chain of supersteps.  Vertex state is laid out [vertex][source] so that
// one 64-lane wavefront holds a vertex's row with lane = source: a vertex's
// sigma row is one coalesced 512-byte read.
//
// Forward: a multi-source BFS superstep (one bit per source in the frontier,
// visited and next masks) discovers level L+1 for every source at once; then
// each newly reached vertex w pulls, for every source s whose frontier
// reached it, sigma[w][s] = sum of sigma[u][s] over in-neighbours u that were
// on s's frontier at level L (the level-L masks are kept until the pull is
// done).  The queue of each level is kept with the mask of each entry.
// Backward: for L from the deepest level down to 1, every vertex v with some
// source at level L computes, per such source,
//   delta[v][s] = sigma[v][s] * sum over out-neighbours w with s at level
//                 L+1 of g[w][s],   g[w][s] = (1 + delta[w][s]) / sigma[w][s]
// (Brandes' recurrence with the child's factor formed once per vertex in
// fp64 and kept in fp32, where one rounding takes the place of the three of
// a ratio, a sum and a product per edge).  The sums run in fp64; a last pass
// adds each vertex's delta row to its score.
//
// Both passes are one operation: per row, the sum of the neighbours' state
// rows, masked by the neighbours' source masks.  It is bound by the rows
// fetched (512 or 256 bytes each, from the L2s and beyond), so the wave that
// sums a row reads 64 neighbours' ids and masks at a time, one per lane,
// drops those with no source in common, and keeps eight state rows in
// flight.  Rows take waves by degree: hubs (the HUB bin) several blocks each
// with partial sums added by a second launch, the BLOCK bin a block, the
// WAVE bin a wave; below that a wave takes several consecutive queue entries
// and walks their edges as one list, because the chain of dependent reads
// (entry, offsets, ids, masks, rows) is otherwise paid per short row.
// RMAT-20, 64 sources: @BC@.
#include <string.h>

#include <algorithm>
#include <vector>

#include "tg_internal.h"

using namespace tgk;

namespace tg {
namespace {

using u64 = unsigned long long;
constexpr int S = 64;  // sources per chain

inline unsigned nblk(int64_t n) { return (unsigned)std::max<int64_t>((n + BLOCK - 1) / BLOCK, 1); }

__global__ __launch_bounds__(BLOCK) void k_bb_expand(const Plan *__restrict__ Pp, const int32_t *__restrict__ queue,
                                                     const int64_t *__restrict__ hubpref,
                                                     const int64_t *__restrict__ off, const int32_t *__restrict__ col,
                                                     const u64 *front, const u64 *visited, u64 *next,
                                                     uint32_t *touched, int64_t hub_chunk) {
  const Plan &P = load_plan(Pp);
  const int64_t total = P.vb[NBIN];
  for (int64_t vb = blockIdx.x; vb < total; vb += gridDim.x) {
    const Assign a = assign_work(vb, P, queue, nullptr, hubpref, off, hub_chunk);
    if (!a.ok) continue;
    const u64 m = front[a.v];
    if (m == 0) continue;
    for (int64_t e = a.e_begin + a.lane; e < a.e_end; e += a.stride) {
      const int32_t nb = stream_load(col + e);
      const u64 x = m & ~visited[nb];
      if (x && atomicOr(next + nb, x) == 0) atomicOr(touched + (nb >> 5), 1u << (nb & 31));
    }
  }
}

template <typename T>
__global__ __launch_bounds__(BLOCK) void k_bb_fill(T *p, int64_t n, T v) {
  for (int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLOCK) p[i] = v;
}

// Settle level L+1: new bits, visited, the new frontier masks and the mask of
// each queue entry.
__global__ __launch_bounds__(BLOCK) void k_bb_finalize(const Plan *__restrict__ Pp, const int32_t *__restrict__ queue,
                                                       u64 *__restrict__ qmask, u64 *visited, u64 *front_new,
                                                       u64 *next) {
  const int32_t count = Pp->count;
  for (int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x; i < count; i += (int64_t)gridDim.x * BLOCK) {
    const int32_t v = queue[i];
    const u64 seen = visited[v];
    const u64 nb = next[v] & ~seen;
    next[v] = 0;
    visited[v] = seen | nb;
    front_new[v] = nb;
    qmask[i] = nb;
  }
}

__device__ __forceinline__ u64 lane_mask(u64 m, int src) {
  return (u64)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)m, src) |
         ((u64)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(m >> 32), src) << 32);
}

__device__ __forceinline__ int64_t lane_i64(int64_t x, int src) { return (int64_t)lane_mask((u64)x, src); }

// The sigma pull: rows are sigma rows (fp64), a row's sum is the vertex's own.
struct SigmaOp {
  using T = double;
  double *rows;
  uint32_t *flags;
  __device__ __forceinline__ double begin(int32_t, u64) const { return 0.0; }
  __device__ __forceinline__ void end(int32_t v, u64 m, double, double acc) const {
    const int lane = threadIdx.x & 63;
    if ((m >> lane) & 1ull) {
      rows[(int64_t)v * S + lane] = acc;
      if (acc >= 9007199254740992.0) flags[2] = 1u;  // 2^53
    }
  }
};

// The dependencies: rows are g rows (fp32).  The vertex's mask at its level
// becomes the child mask of the next pass.
struct DeltaOp {
  using T = float;
  float *rows;
  const double *sigma;
  float *delta;
  u64 *mask_out;
  __device__ __forceinline__ double begin(int32_t v, u64 m) const {
    const int lane = threadIdx.x & 63;
    return (m >> lane) & 1ull ? sigma[(int64_t)v * S + lane] : 1.0;
  }
  __device__ __forceinline__ void end(int32_t v, u64 m, double sv, double acc) const {
    const int lane = threadIdx.x & 63;
    if ((m >> lane) & 1ull) {
      const float d = (float)(sv * acc);
      delta[(int64_t)v * S + lane] = d;
      rows[(int64_t)v * S + lane] = (float)((1.0 + (double)d) / sv);
    }
    if (lane == 0) mask_out[v] = m;
  }
};

constexpr int FLY = 8;  // state rows in flight per wave

// Sum, over the tiles of 64 edges first, first + step, ... of [e0, e1), of
// the neighbours' rows masked by mask[u] & m (lane = source).
template <typename T>
__device__ __forceinline__ double masked_rows(const int32_t *__restrict__ col, int64_t e0, int64_t e1, int first,
                                              int step, const u64 *__restrict__ mask, u64 m, const T *rows) {
  const int lane = threadIdx.x & 63;
  const int64_t stride = (int64_t)step * 64;
  double acc = 0.0;
  int64_t e = e0 + (int64_t)first * 64;
  int32_t u = e + lane < e1 ? stream_load(col + e + lane) : -1;
  while (e < e1) {
    const u64 mu = u >= 0 ? mask[u] & m : 0ull;
    const int32_t uc = u;
    e += stride;
    u = e + lane < e1 ? stream_load(col + e + lane) : -1;  // the next tile's ids
    for (u64 todo = __ballot(mu != 0ull); todo;) {
      T x[FLY];
#pragma unroll
      for (int k = 0; k < FLY; ++k) {
        x[k] = (T)0;
        if (todo) {
          const int src = __ffsll((long long)todo) - 1;
          todo &= todo - 1;
          if ((lane_mask(mu, src) >> lane) & 1ull)
            x[k] = rows[(int64_t)__builtin_amdgcn_readlane(uc, src) * S + lane];
        }
      }
#pragma unroll
      for (int k = 0; k < FLY; ++k) acc += (double)x[k];
    }
  }
  return acc;
}

// Sum of the block's four waves' per-lane partials (every wave gets it).
__device__ __forceinline__ double block_lane_sum(double x) {
  __shared__ double red[BLOCK];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  __syncthreads();
  red[w * 64 + lane] = x;
  __syncthreads();
  return red[lane] + red[64 + lane] + red[128 + lane] + red[192 + lane];
}

// The BLOCK bin: queue entries [lo, hi), a block each.
template <class Op>
__global__ __launch_bounds__(BLOCK) void k_bb_block(const int32_t *__restrict__ queue, const u64 *__restrict__ qmask,
                                                    int32_t lo, int32_t hi, const int64_t *__restrict__ off,
                                                    const int32_t *__restrict__ col, const u64 *__restrict__ mask,
                                                    Op op) {
  const int w = threadIdx.x >> 6;
  for (int64_t i = lo + (int64_t)blockIdx.x; i < hi; i += gridDim.x) {
    const int32_t v = queue[i];
    const u64 m = qmask[i];  // block-uniform, never 0
    const double pre = op.begin(v, m);
    const double acc = block_lane_sum(masked_rows(col, off[v], off[v + 1], w, BLOCK / 64, mask, m, op.rows));
    if (w == 0) op.end(v, m, pre, acc);
  }
}

// The HUB bin: queue entries [0, hubs), gridDim.y blocks each; block y of
// entry i leaves its share in part[i * gridDim.y + y].
template <class Op>
__global__ __launch_bounds__(BLOCK) void k_bb_hubs(const int32_t *__restrict__ queue, const u64 *__restrict__ qmask,
                                                   int32_t hubs, const int64_t *__restrict__ off,
                                                   const int32_t *__restrict__ col, const u64 *__restrict__ mask,
                                                   Op op, double *__restrict__ part) {
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int64_t i = blockIdx.x; i < hubs; i += gridDim.x) {
    const int32_t v = queue[i];
    const u64 m = qmask[i];
    const double acc = block_lane_sum(masked_rows(col, off[v], off[v + 1], (int)blockIdx.y * (BLOCK / 64) + w,
                                                  (int)gridDim.y * (BLOCK / 64), mask, m, op.rows));
    if (w == 0) part[(i * gridDim.y + blockIdx.y) * S + lane] = acc;
  }
}

// One wave per hub adds its shares in order and finishes the row.
template <class Op>
__global__ __launch_bounds__(BLOCK) void k_bb_hubs_finish(const int32_t *__restrict__ queue,
                                                          const u64 *__restrict__ qmask, int32_t hubs, int shares,
                                                          const double *__restrict__ part, Op op) {
  const int lane = threadIdx.x & 63;
  const int64_t i = ((int64_t)blockIdx.x * BLOCK + threadIdx.x) >> 6;
  if (i >= hubs) return;
  const int32_t v = queue[i];
  const u64 m = qmask[i];
  const double pre = op.begin(v, m);
  double acc = 0.0;
  for (int y = 0; y < shares; ++y) acc += part[(i * shares + y) * S + lane];
  op.end(v, m, pre, acc);
}

// Queue entries [i0, i0 + k), k <= 64, by one wave.  Lane j holds entry j;
// the entries' edges are walked as one list, 64 at a time, each lane finding
// the entry its edge belongs to from the entries' first positions in the
// list.  Edges stay in order, so a row's sum is finished when the owner of
// the next contributing edge is another entry.
template <class Op>
__device__ __forceinline__ void rows_of_entries(const int32_t *__restrict__ queue, const u64 *__restrict__ qmask,
                                                int64_t i0, int k, const int64_t *__restrict__ off,
                                                const int32_t *__restrict__ col, const u64 *__restrict__ mask,
                                                const Op &op) {
  using T = typename Op::T;
  const int lane = threadIdx.x & 63;
  int32_t v = 0;
  u64 m = 0;
  int64_t e0 = 0, d = 0;
  if (lane < k) {
    v = queue[i0 + lane];
    m = qmask[i0 + lane];
    e0 = off[v];
    d = off[v + 1] - e0;
  }
  // first list position of each entry, and the list's length
  int64_t inc = d;
  for (int o = 1; o < 64; o <<= 1) {
    const int64_t y = __shfl_up((long long)inc, o, 64);
    if (lane >= o) inc += y;
  }
  const int64_t total = lane_i64(inc, 63);
  if (k == 1 || total >= ((int64_t)1 << 30)) {
    // one entry (or rows too long for 32-bit positions): row by row
    for (int j = 0; j < k; ++j) {
      const int32_t vj = __builtin_amdgcn_readlane(v, j);
      const u64 mj = lane_mask(m, j);
      const int64_t ej = lane_i64(e0, j);
      const double pre = op.begin(vj, mj);
      op.end(vj, mj, pre, masked_rows(col, ej, ej + lane_i64(d, j), 0, 1, mask, mj, op.rows));
    }
    return;
  }
  const int32_t start = (int32_t)(inc - d), len = (int32_t)total;
  int span = 1;  // search steps: the least power of two >= k
  while (span < k) span <<= 1;
  int cur = -1;
  double acc = 0.0, pre = 0.0;
  u64 open = __ballot(lane < k);
  const auto finish = [&]() {
    op.end(__builtin_amdgcn_readlane(v, cur), lane_mask(m, cur), pre, acc);
    open &= ~(1ull << cur);
  };
  for (int32_t t0 = 0; t0 < len; t0 += 64) {
    const int32_t t = t0 + lane;
    int own = 0;
    for (int h = span >> 1; h > 0; h >>= 1) {
      const int32_t s = __shfl(start, own + h, 64);
      if (own + h < k && s <= t) own += h;
    }
    const int64_t eo = __shfl((long long)e0, own, 64);
    const int32_t so = __shfl(start, own, 64);
    const u64 mo = (u64)__shfl((long long)m, own, 64);
    int32_t u = -1;
    u64 mu = 0;
    if (t < len) {
      u = stream_load(col + eo + (t - so));
      mu = mask[u] & mo;
    }
    for (u64 todo = __ballot(mu != 0ull); todo;) {
      T x[FLY];
      double p[FLY];
      int o[FLY];
      int prev = cur;
#pragma unroll
      for (int q = 0; q < FLY; ++q) {
        x[q] = (T)0;
        p[q] = 0.0;
        o[q] = -1;
        if (todo) {
          const int src = __ffsll((long long)todo) - 1;
          todo &= todo - 1;
          o[q] = __builtin_amdgcn_readlane(own, src);
          if (o[q] != prev)
            p[q] = op.begin(__builtin_amdgcn_readlane(v, o[q]), lane_mask(m, o[q]));
          prev = o[q];
          if ((lane_mask(mu, src) >> lane) & 1ull)
            x[q] = op.rows[(int64_t)__builtin_amdgcn_readlane(u, src) * S + lane];
        }
      }
#pragma unroll
      for (int q = 0; q < FLY; ++q)
        if (o[q] >= 0) {
          if (o[q] != cur) {
            if (cur >= 0) finish();
            cur = o[q];
            pre = p[q];
            acc = 0.0;
          }
          acc += (double)x[q];
        }
    }
  }
  if (cur >= 0) finish();
  // entries no neighbour contributes to (the backward pass: no child)
  while (open) {
    cur = __ffsll((long long)open) - 1;
    pre = op.begin(__builtin_amdgcn_readlane(v, cur), lane_mask(m, cur));
    acc = 0.0;
    finish();
  }
}

// The bins below BLOCK: queue entries [p0, p1) (WAVE bin) one to a wave,
// [p1, p2) (G16) G16_ROWS to a wave, [p2, p3) (the rest) LOW_ROWS to a wave.
constexpr int G16_ROWS = 4, LOW_ROWS = 16;
template <class Op>
__global__ __launch_bounds__(BLOCK) void k_bb_rows(const int32_t *__restrict__ queue, const u64 *__restrict__ qmask,
                                                   int64_t p0, int64_t p1, int64_t p2, int64_t p3,
                                                   const int64_t *__restrict__ off, const int32_t *__restrict__ col,
                                                   const u64 *__restrict__ mask, Op op) {
  const int64_t w1 = p1 - p0, w2 = w1 + (p2 - p1 + G16_ROWS - 1) / G16_ROWS,
                w3 = w2 + (p3 - p2 + LOW_ROWS - 1) / LOW_ROWS;
  const int64_t nw = ((int64_t)gridDim.x * BLOCK) >> 6;
  const int64_t mine = ((int64_t)blockIdx.x * BLOCK + threadIdx.x) >> 6;
  for (int64_t x = mine; x < w3; x += nw) {
    // wave-uniform: entries [i, i + k)
    const int64_t w = lane_i64(x, 0);
    int64_t i, end;
    int k;
    if (w < w1) {
      i = p0 + w;
      k = 1;
      end = p1;
    } else if (w < w2) {
      i = p1 + (w - w1) * G16_ROWS;
      k = G16_ROWS;
      end = p2;
    } else {
      i = p2 + (w - w2) * LOW_ROWS;
      k = LOW_ROWS;
      end = p3;
    }
    if (i + k > end) k = (int)(end - i);
    rows_of_entries(queue, qmask, i, k, off, col, mask, op);
  }
}

// The deepest level: delta is 0, so g = 1 / sigma; its masks start the
// backward pass.
__global__ __launch_bounds__(BLOCK) void k_bb_deepest(const int32_t *__restrict__ queue,
                                                      const u64 *__restrict__ qmask, int32_t count, DeltaOp op) {
  const int64_t nw = ((int64_t)gridDim.x * BLOCK) >> 6;
  for (int64_t i = ((int64_t)blockIdx.x * BLOCK + threadIdx.x) >> 6; i < count; i += nw) {
    const int32_t v = queue[i];
    const u64 m = qmask[i];
    op.end(v, m, op.begin(v, m), 0.0);
  }
}

// score[v] += the vertex's delta row: 16 lanes a row, four sources a lane.
__global__ __launch_bounds__(BLOCK) void k_bb_score(const float4 *__restrict__ delta, int64_t n,
                                                    double *__restrict__ score) {
  const int64_t t = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  const int64_t v = t >> 4;
  double x = 0.0;
  if (v < n) {
    const float4 d = delta[t];
    x = ((double)d.x + (double)d.y) + ((double)d.z + (double)d.w);
  }
  x = group_sum(x, 16);
  if (v < n && (t & 15) == 0 && x != 0.0) score[v] += x;
}

struct Roots {
  int32_t v[S];
};

// The sources join: their bit on the next masks, sigma 1.
__global__ __launch_bounds__(S) void k_bb_join(u64 *next, uint32_t *touched, double *sigma, Roots roots, int count) {
  const int k = threadIdx.x;
  if (k >= count) return;
  const int32_t r = roots.v[k];
  atomicOr(next + r, 1ull << k);
  atomicOr(touched + (r >> 5), 1u << (r & 31));
  sigma[(int64_t)r * S + k] = 1.0;
}

// Blocks that share a hub's row: as many as the partial sums' room allows
// (part_rows of them), 16 at most.
int hub_shares(int64_t part_rows, int32_t hubs) {
  return (int)std::max<int64_t>(1, std::min<int64_t>(part_rows / hubs, 16));
}

// One pass over a level's queue (plan P): rows of off / col, masks `mask`.
template <class Op>
int launch_rows(const Plan &P, const int32_t *queue, const u64 *qmask, const int64_t *off, const int32_t *col,
                const u64 *mask, const Op &op, double *part, int64_t part_rows, hipStream_t s) {
  const int32_t hubs = P.pos[1], split = P.pos[BIN_WAVE], count = P.count;
  if (hubs > 0) {
    const int shares = hub_shares(part_rows, hubs);
    hipLaunchKernelGGL(k_bb_hubs<Op>, dim3((unsigned)std::min<int32_t>(hubs, 16384), (unsigned)shares), dim3(BLOCK), 0,
                       s, queue, qmask, hubs, off, col, mask, op, part);
    hipLaunchKernelGGL(k_bb_hubs_finish<Op>, dim3((unsigned)((hubs + 3) / 4)), dim3(BLOCK), 0, s, queue, qmask, hubs,
                       shares, part, op);
  }
  if (split > hubs)
    hipLaunchKernelGGL(k_bb_block<Op>, dim3((unsigned)std::min<int32_t>(split - hubs, 16384)), dim3(BLOCK), 0, s,
                       queue, qmask, hubs, split, off, col, mask, op);
  if (count > split) {
    const int64_t p1 = P.pos[BIN_G16], p2 = P.pos[BIN_G4];
    const int64_t waves = (p1 - split) + (p2 - p1 + G16_ROWS - 1) / G16_ROWS + (count - p2 + LOW_ROWS - 1) / LOW_ROWS;
    hipLaunchKernelGGL(k_bb_rows<Op>, dim3((unsigned)std::min<int64_t>((waves + 3) / 4, 32768)), dim3(BLOCK), 0, s,
                       queue, qmask, (int64_t)split, p1, p2, (int64_t)count, off, col, mask, op);
  }
  TG_HIP(hipGetLastError());
  return TG_OK;
}

}  // namespace

// Scratch of the batched BC (lazy, per partition).
struct BcBatchState {
  DevArena arena;
  Workspace ws;
  int64_t n = -1;
  u64 *masks = nullptr;                // visited, front[0], front[1], next back to back
  u64 *visited = nullptr, *front[2] = {nullptr, nullptr}, *next = nullptr;
  double *sigma = nullptr;
  float *delta = nullptr, *g = nullptr;
  int32_t *queue_all = nullptr;  // level queues back to back
  u64 *qmask = nullptr;          // the mask of each queue entry
  int64_t qcap = 0;              // entries there is room for
  double *hub_part = nullptr;    // hubs' partial sums, a row of S each
  int64_t part_rows = 0;

  // Room for `need` queue entries, keeping the first `used`.
  int grow(int64_t need, int64_t used, hipStream_t s) {
    if (need <= qcap) return TG_OK;
    const int64_t cap = std::max(need, 2 * qcap);
    int32_t *q = nullptr;
    u64 *m = nullptr;
    TG_TRY(dalloc(arena, &q, (size_t)cap));
    TG_TRY(dalloc(arena, &m, (size_t)cap));
    if (used > 0) {
      TG_HIP(hipMemcpyAsync(q, queue_all, (size_t)used * sizeof(int32_t), hipMemcpyDeviceToDevice, s));
      TG_HIP(hipMemcpyAsync(m, qmask, (size_t)used * sizeof(u64), hipMemcpyDeviceToDevice, s));
      TG_HIP(hipStreamSynchronize(s));
    }
    if (queue_all) {
      arena.release_one(queue_all);
      arena.release_one(qmask);
    }
    queue_all = q;
    qmask = m;
    qcap = cap;
    return TG_OK;
  }
};

void bcb_free(tg_partition *p) {
  delete p->bcb;
  p->bcb = nullptr;
}

int gpu_bc_batched(tg_partition *p, const int32_t *sources, int32_t ns, hipStream_t s) {
  GpuPart &g = p->gpu;
  const Tuning &t = p->tune;
  if (!p->bcb) {
    p->bcb = new (std::nothrow) BcBatchState();
    if (!p->bcb) return set_error(TG_ENOMEM, "bc_batched: out of host memory");
  }
  BcBatchState &B = *p->bcb;
  const int64_t n = std::max<int64_t>(g.n, 1);
  TG_TRY(B.ws.ensure(g, 0));
  if (B.n != g.n || B.part_rows < g.max_out_hubs) {
    B.n = -1;
    B.arena.release();
    B.queue_all = nullptr;
    B.qmask = nullptr;
    B.qcap = 0;
    TG_TRY(dalloc(B.arena, &B.masks, (size_t)n * 4));
    B.visited = B.masks;
    B.front[0] = B.masks + n;
    B.front[1] = B.masks + 2 * n;
    B.next = B.masks + 3 * n;
    TG_TRY(dalloc(B.arena, &B.sigma, (size_t)n * S));
    TG_TRY(dalloc(B.arena, &B.delta, (size_t)n * S));
    TG_TRY(dalloc(B.arena, &B.g, (size_t)n * S));
    // a vertex is queued once per level that some source reaches it at: a
    // few times on graphs of small depth (more room is made when needed)
    TG_TRY(B.grow(6 * n, 0, s));
    // at least one partial sum per hub; 256 edges and more per share
    B.part_rows = g.m / 256 + g.max_out_hubs + 1;
    TG_TRY(dalloc(B.arena, &B.hub_part, (size_t)B.part_rows * S));
    B.n = g.n;
  }
  Workspace &ws = B.ws;
  const unsigned fill_grid = 4096;
  TG_HIP(hipMemsetAsync(ws.counters, 0, 4 * sizeof(uint32_t), s));  // an earlier call's overflow flag
  for (int32_t c0 = 0; c0 < ns; c0 += S) {
    const int32_t cn = std::min<int32_t>(S, ns - c0);
    TG_HIP(hipMemsetAsync(B.masks, 0, (size_t)n * 4 * sizeof(u64), s));
    TG_HIP(hipMemsetAsync(ws.bits_a, 0, ws.nwords * sizeof(uint32_t), s));
    hipLaunchKernelGGL(k_bb_fill<float4>, dim3(fill_grid), dim3(BLOCK), 0, s, reinterpret_cast<float4 *>(B.delta),
                       n * S / 4, make_float4(0.f, 0.f, 0.f, 0.f));
    Roots roots;
    for (int32_t k = 0; k < cn; ++k) roots.v[k] = p->h_l_of_g[sources[c0 + k]];
    hipLaunchKernelGGL(k_bb_join, dim3(1), dim3(S), 0, s, B.next, ws.bits_a, B.sigma, roots, (int)cn);
    TG_HIP(hipGetLastError());
    // level 0: the sources
    std::vector<Plan> plans;
    std::vector<int64_t> segoff;
    int64_t off = 0;
    int cur = 0;
    TG_TRY(frontier_compact(g, ws, 1, ws.bits_a, nullptr, B.queue_all, nullptr, 0, s));
    TG_TRY(frontier_plan(g, ws, B.queue_all, t, s, false));
    hipLaunchKernelGGL(k_bb_finalize, dim3(1), dim3(BLOCK), 0, s, ws.plan, B.queue_all, B.qmask, B.visited,
                       B.front[cur], B.next);
    TG_HIP(hipMemcpyAsync(ws.h_plan, ws.plan, sizeof(Plan), hipMemcpyDeviceToHost, s));
    TG_HIP(hipStreamSynchronize(s));
    int32_t L = 0;
    for (;;) {
      if (L > g.n) return set_error(TG_EDEVICE, "bc_batched: more supersteps than vertices");
      const Plan P = *ws.h_plan;
      plans.push_back(P);
      segoff.push_back(off);
      const int64_t noff = off + P.count;
      TG_TRY(B.grow(noff + n, noff, s));
      if (P.vb[NBIN] > 0)
        hipLaunchKernelGGL(k_bb_expand, dim3(launch_grid(P.vb[NBIN])), dim3(BLOCK), 0, s, ws.plan, B.queue_all + off,
                           ws.hubpref, g.out.off, g.out.col, B.front[cur], B.visited, B.next, ws.bits_a,
                           t.hub_chunk);
      TG_TRY(frontier_compact(g, ws, 1, ws.bits_a, nullptr, B.queue_all + noff, nullptr, 0, s));
      TG_TRY(frontier_plan(g, ws, B.queue_all + noff, t, s, false));
      hipLaunchKernelGGL(k_bb_finalize, dim3(nblk(std::min<int64_t>(n, 1 << 20))), dim3(BLOCK), 0, s, ws.plan,
                         B.queue_all + noff, B.qmask + noff, B.visited, B.front[cur ^ 1], B.next);
      TG_HIP(hipMemcpyAsync(ws.h_plan, ws.plan, sizeof(Plan), hipMemcpyDeviceToHost, s));
      TG_HIP(hipStreamSynchronize(s));
      TG_HIP(hipGetLastError());
      if (ws.h_plan->count == 0) break;
      const int tk = ktimer_start(s);
      TG_TRY(launch_rows(*ws.h_plan, B.queue_all + noff, B.qmask + noff, g.in.off, g.in.col, B.front[cur],
                         SigmaOp{B.sigma, ws.counters}, B.hub_part, B.part_rows, s));
      ktimer_stop(tk, s, "bcb_sigma");
      TG_HIP(hipMemsetAsync(B.front[cur], 0, (size_t)n * sizeof(u64), s));
      cur ^= 1;
      off = noff;
      ++L;
    }
    if (L > 1) {
      // backward: level L is the deepest reached; its dependencies stay 0
      u64 *child = B.front[0], *own = B.front[1];
      TG_HIP(hipMemsetAsync(B.front[0], 0, (size_t)n * 2 * sizeof(u64), s));
      hipLaunchKernelGGL(k_bb_deepest, dim3((unsigned)std::min<int64_t>((plans[L].count + 3) / 4, 16384)), dim3(BLOCK),
                         0, s, B.queue_all + segoff[L], B.qmask + segoff[L], plans[L].count,
                         DeltaOp{B.g, B.sigma, B.delta, child});
      for (int32_t lv = L - 1; lv >= 1; --lv) {
        const int tk = ktimer_start(s);
        TG_TRY(launch_rows(plans[lv], B.queue_all + segoff[lv], B.qmask + segoff[lv], g.out.off, g.out.col, child,
                           DeltaOp{B.g, B.sigma, B.delta, own}, B.hub_part, B.part_rows, s));
        ktimer_stop(tk, s, "bcb_delta");
        TG_HIP(hipMemsetAsync(child, 0, (size_t)n * sizeof(u64), s));
        std::swap(child, own);
      }
      hipLaunchKernelGGL(k_bb_score, dim3((unsigned)((g.n * 16 + BLOCK - 1) / BLOCK)), dim3(BLOCK), 0, s,
                         reinterpret_cast<const float4 *>(B.delta), g.n, p->ws.bc_acc);
      TG_HIP(hipGetLastError());
    }
    TG_HIP(hipMemcpyAsync(ws.h_flags, ws.counters, 4 * sizeof(uint32_t), hipMemcpyDeviceToHost, s));
    TG_HIP(hipStreamSynchronize(s));
    if (ws.h_flags[2]) return set_error(TG_ERANGE, "bc_batched: a shortest-path count reached 2^53");
  }
  return TG_OK;
}

}  // namespace tg
