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
// WAVE bin a wave, and these two bins several blocks too where a level has
// few of them; below that a wave takes several consecutive queue entries and
// walks their edges as one list (the walks are in ms.h).
// RMAT-20, 64 sources: 23.6 ms a call with four edges in flight per wave and
// three rows (level, sigma, delta) read per edge, 6.9 so, 6.1 with the
// levels pulled (ms.hip) where 970 us of pushes had been, 5.9 with few rows
// shared.
#include <string.h>

#include <algorithm>
#include <vector>

#include "ms.h"

using namespace tgk;

namespace tg {
namespace {

constexpr int S = kSlots;  // sources per chain

inline unsigned nblk(int64_t n) { return (unsigned)std::max<int64_t>((n + BLOCK - 1) / BLOCK, 1); }

template <typename T>
__global__ __launch_bounds__(BLOCK) void k_bb_fill(T *p, int64_t n, T v) {
  for (int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLOCK) p[i] = v;
}

// Settle level L+1: new bits, visited, the new frontier masks, the mask of
// each queue entry and the frontier's edges per source.
__global__ __launch_bounds__(BLOCK) void k_bb_finalize(const Plan *__restrict__ Pp, const int32_t *__restrict__ queue,
                                                       u64 *__restrict__ qmask, u64 *visited, u64 *front_new,
                                                       u64 *next, const int64_t *__restrict__ off,
                                                       u64 (*mf)[kSlots], u64 (*other)[kSlots]) {
  const int32_t count = Pp->count;
  u64 acc = 0;
  for (int64_t b = (int64_t)blockIdx.x * BLOCK; b < count; b += (int64_t)gridDim.x * BLOCK) {
    const int64_t i = b + threadIdx.x;
    u64 nb = 0;
    uint32_t edges = 0;
    if (i < count) {
      const int32_t v = queue[i];
      const u64 seen = visited[v];
      nb = next[v] & ~seen;
      next[v] = 0;
      visited[v] = seen | nb;
      front_new[v] = nb;
      qmask[i] = nb;
      edges = (uint32_t)(off[v + 1] - off[v]) + 1u;
    }
    add_by_slot(nb, edges, acc);
  }
  publish_by_slot<BLOCK>(acc, mf, other);
}

// The sigma pull: rows are sigma rows (fp64), a row's sum is the vertex's own.
struct SigmaOp {
  using X = double;
  using A = double;
  using P = double;
  static constexpr bool WEIGHTS = false;
  double *rows;
  uint32_t *flags;
  __device__ __forceinline__ A zero() const { return 0.0; }
  __device__ __forceinline__ P begin(int32_t, u64) const { return 0.0; }
  __device__ __forceinline__ X load(int32_t u, u64 m) const {
    const int lane = threadIdx.x & 63;
    return (m >> lane) & 1ull ? rows[(int64_t)u * S + lane] : 0.0;
  }
  __device__ __forceinline__ void add(A &acc, X x, int32_t) const { acc += x; }
  __device__ __forceinline__ void end(int, int32_t v, u64 m, P, A acc) const {
    const int lane = threadIdx.x & 63;
    if ((m >> lane) & 1ull) {
      rows[(int64_t)v * S + lane] = acc;
      if (acc >= 9007199254740992.0) flags[2] = 1u;  // 2^53
    }
  }
  __device__ __forceinline__ void idle(int32_t, u64, u64) const {}  // (a reached vertex has a parent)
};

// The dependencies: rows are g rows (fp32).  The vertex's mask at its level
// becomes the child mask of the next pass.
struct DeltaOp {
  using X = float;
  using A = double;
  using P = double;
  static constexpr bool WEIGHTS = false;
  float *rows;
  const double *sigma;
  float *delta;
  u64 *mask_out;
  __device__ __forceinline__ A zero() const { return 0.0; }
  __device__ __forceinline__ P begin(int32_t v, u64 m) const {
    const int lane = threadIdx.x & 63;
    return (m >> lane) & 1ull ? sigma[(int64_t)v * S + lane] : 1.0;
  }
  __device__ __forceinline__ X load(int32_t u, u64 m) const {
    const int lane = threadIdx.x & 63;
    return (m >> lane) & 1ull ? rows[(int64_t)u * S + lane] : 0.0f;
  }
  __device__ __forceinline__ void add(A &acc, X x, int32_t) const { acc += (double)x; }
  __device__ __forceinline__ void end(int, int32_t v, u64 m, P sv, A acc) const {
    const int lane = threadIdx.x & 63;
    if ((m >> lane) & 1ull) {
      const float d = (float)(sv * acc);
      delta[(int64_t)v * S + lane] = d;
      rows[(int64_t)v * S + lane] = (float)((1.0 + (double)d) / sv);
    }
    if (lane == 0) mask_out[v] = m;
  }
  // no child: delta is 0
  __device__ __forceinline__ void idle(int32_t v, u64 m, u64 open) const {
    for (; open; open &= open - 1) {
      const int j = __ffsll((long long)open) - 1;
      const int32_t vj = __builtin_amdgcn_readlane(v, j);
      const u64 mj = lane_mask(m, j);
      end(j, vj, mj, begin(vj, mj), 0.0);
    }
  }
};

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
    const double acc = block_lane_sum(walk_row(op, col, off[v], off[v + 1], w, BLOCK / 64, mask, m));
    if (w == 0) op.end(0, v, m, pre, acc);
  }
}

// Rows of queue entries [0, rows), gridDim.y blocks each; block y of entry i
// leaves its share in part[i * gridDim.y + y].
template <class Op>
__global__ __launch_bounds__(BLOCK) void k_bb_shared(const int32_t *__restrict__ queue, const u64 *__restrict__ qmask,
                                                   int32_t rows, const int64_t *__restrict__ off,
                                                   const int32_t *__restrict__ col, const u64 *__restrict__ mask,
                                                   Op op, double *__restrict__ part) {
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int64_t i = blockIdx.x; i < rows; i += gridDim.x) {
    const int32_t v = queue[i];
    const u64 m = qmask[i];
    const double acc = block_lane_sum(walk_row(op, col, off[v], off[v + 1], (int)blockIdx.y * (BLOCK / 64) + w,
                                               (int)gridDim.y * (BLOCK / 64), mask, m));
    if (w == 0) part[(i * gridDim.y + blockIdx.y) * S + lane] = acc;
  }
}

// One wave per row adds its shares in order, eight reads in flight, and
// finishes the row.
template <class Op>
__global__ __launch_bounds__(BLOCK) void k_bb_shared_finish(const int32_t *__restrict__ queue,
                                                          const u64 *__restrict__ qmask, int32_t rows, int shares,
                                                          const double *__restrict__ part, Op op) {
  const int lane = threadIdx.x & 63;
  const int64_t i = ((int64_t)blockIdx.x * BLOCK + threadIdx.x) >> 6;
  if (i >= rows) return;
  const int32_t v = queue[i];
  const u64 m = qmask[i];
  const double pre = op.begin(v, m);
  double acc = 0.0;
  for (int y = 0; y < shares; y += 8) {
    double x[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) x[q] = y + q < shares ? part[(i * shares + y + q) * S + lane] : 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q) acc += x[q];
  }
  op.end(0, v, m, pre, acc);
}

// The bins below BLOCK: queue entries of the spans R.
template <class Op>
__global__ __launch_bounds__(BLOCK) void k_bb_rows(const int32_t *__restrict__ queue, const u64 *__restrict__ qmask,
                                                   RowSpans R, const int64_t *__restrict__ off,
                                                   const int32_t *__restrict__ col, const u64 *__restrict__ mask,
                                                   Op op) {
  for_row_spans(R, ((int64_t)blockIdx.x * BLOCK + threadIdx.x) >> 6, ((int64_t)gridDim.x * BLOCK) >> 6,
                [&](int64_t i, int k) {
                  Entries E;
                  E.load([&](int64_t x) { return queue[x]; }, [&](int64_t x, int32_t) { return qmask[x]; }, i, k, off);
                  walk_list(op, E, col, mask);
                });
}

// The deepest level: delta is 0, so g = 1 / sigma; its masks start the
// backward pass.
__global__ __launch_bounds__(BLOCK) void k_bb_deepest(const int32_t *__restrict__ queue,
                                                      const u64 *__restrict__ qmask, int32_t count, DeltaOp op) {
  const int64_t nw = ((int64_t)gridDim.x * BLOCK) >> 6;
  for (int64_t i = ((int64_t)blockIdx.x * BLOCK + threadIdx.x) >> 6; i < count; i += nw) {
    const int32_t v = queue[i];
    const u64 m = qmask[i];
    op.end(0, v, m, op.begin(v, m), 0.0);
  }
}

// score[v] += the vertex's delta row: 16 lanes a row, four sources a lane.
__global__ __launch_bounds__(BLOCK) void k_bb_score(const float4 *__restrict__ delta, int64_t n,
                                                    double *__restrict__ score) {
  // (a row's 16 lanes are in the loop together)
  for (int64_t t = (int64_t)blockIdx.x * BLOCK + threadIdx.x; t < n * 16; t += (int64_t)gridDim.x * BLOCK) {
    const float4 d = delta[t];
    const double x = group_sum(((double)d.x + (double)d.y) + ((double)d.z + (double)d.w), 16);
    if ((t & 15) == 0 && x != 0.0) score[t >> 4] += x;
  }
}

struct Sources {
  int32_t v[S];
};

// The sources join: their bit on the next masks, sigma 1.
__global__ __launch_bounds__(S) void k_bb_join(u64 *next, uint32_t *touched, double *sigma, Sources roots, int count) {
  const int k = threadIdx.x;
  if (k >= count) return;
  const int32_t r = roots.v[k];
  atomicOr(next + r, 1ull << k);
  atomicOr(touched + (r >> 5), 1u << (r & 31));
  sigma[(int64_t)r * S + k] = 1.0;
}

// Blocks that share each of `rows` rows: enough for the chip, as many as
// `most` (a wave's tile of 64 edges each, 16 in any case for hubs) and as the
// partial sums have room for.
int row_shares(int64_t part_rows, int32_t rows, int least, int most) {
  const int64_t want = std::max<int64_t>(least, std::min<int64_t>(2048 / rows, most));
  return (int)std::max<int64_t>(1, std::min<int64_t>(part_rows / rows, want));
}

// Rows of queue entries [lo, hi), `shares` blocks each.
template <class Op>
int launch_shared(int32_t lo, int32_t hi, int shares, int64_t part_rows, const int32_t *queue, const u64 *qmask,
                  const int64_t *off, const int32_t *col, const u64 *mask, const Op &op, double *part, hipStream_t s) {
  const int32_t rows = hi - lo;
  if ((int64_t)rows * shares > part_rows)
    return set_error(TG_EDEVICE, "bc_batched: %d rows in %d shares, room for %lld", rows, shares, (long long)part_rows);
  hipLaunchKernelGGL(k_bb_shared<Op>, dim3((unsigned)std::min<int32_t>(rows, 16384), (unsigned)shares), dim3(BLOCK), 0,
                     s, queue + lo, qmask + lo, rows, off, col, mask, op, part);
  hipLaunchKernelGGL(k_bb_shared_finish<Op>, dim3((unsigned)((rows + 3) / 4)), dim3(BLOCK), 0, s, queue + lo,
                     qmask + lo, rows, shares, part, op);
  return TG_OK;
}

// One pass over a level's queue (plan P): rows of off / col, masks `mask`.
// The rows of a bin whose level holds few are shared by several blocks like
// the hubs', as a wave's edges are a chain of dependent reads.  RMAT-18, 4
// sources: 10 hubs 53 us in 16 shares, 19 in 64; 113 rows of the BLOCK bin 122
// us a block each, 19 in 18 shares with their second launch; 78 rows of the
// WAVE bin 50 us a wave each, 14 so; the call 1.64 -> 1.44 ms (lines at half
// or twice the rows: the same).  RMAT-20, 64 sources: 6.44 -> 6.18 ms.
constexpr int32_t SHARED_BLOCK_ROWS = 512, SHARED_WAVE_ROWS = 1024;

template <class Op>
int launch_rows(const Plan &P, const int32_t *queue, const u64 *qmask, const int64_t *off, const int32_t *col,
                const u64 *mask, const Op &op, double *part, int64_t part_rows, hipStream_t s) {
  const int32_t hubs = P.pos[1], split = P.pos[BIN_WAVE], count = P.count;
  int32_t done = 0;
  const auto shared = [&](int32_t hi, int least, int most) -> int {
    const int shares = row_shares(part_rows, hi - done, least, most);
    TG_TRY(launch_shared(done, hi, shares, part_rows, queue, qmask, off, col, mask, op, part, s));
    done = hi;
    return TG_OK;
  };
  // (the partial sums have room for the hubs, but not for any bin's rows)
  const auto few = [&](int32_t rows, int32_t most) {
    return rows > 0 && rows <= most && 2 * (int64_t)rows <= part_rows;
  };
  if (hubs > 0) TG_TRY(shared(hubs, 16, 64));
  if (split > hubs) {
    if (few(split - hubs, SHARED_BLOCK_ROWS)) {
      TG_TRY(shared(split, 1, 32));
    } else {
      hipLaunchKernelGGL(k_bb_block<Op>, dim3((unsigned)std::min<int32_t>(split - hubs, 16384)), dim3(BLOCK), 0, s,
                         queue, qmask, hubs, split, off, col, mask, op);
      done = split;
    }
  }
  if (few(P.pos[BIN_G16] - split, SHARED_WAVE_ROWS)) TG_TRY(shared(P.pos[BIN_G16], 1, 2));
  if (count > done) {
    const RowSpans R{done, P.pos[BIN_G16], P.pos[BIN_G4], count};
    hipLaunchKernelGGL(k_bb_rows<Op>, dim3((unsigned)std::min<int64_t>((R.waves() + 3) / 4, 32768)), dim3(BLOCK), 0, s,
                       queue, qmask, R, off, col, mask, op);
  }
  TG_HIP(hipGetLastError());
  return TG_OK;
}

}  // namespace

// Scratch of the batched BC (lazy, per partition).
struct BcBatchState {
  DevArena arena;
  Workspace ws;
  MsState *state = nullptr, *h_state = nullptr;  // device (its plan takes the place of ws.plan) and pinned copy
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

  ~BcBatchState() {
    if (h_state) TG_QUIET(hipHostFree(h_state));
  }
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
    TG_TRY(dalloc(B.arena, &B.state, 1));
    if (!B.h_state) TG_HIP(hipHostMalloc((void **)&B.h_state, sizeof(MsState), hipHostMallocDefault));
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
  ws.plan = &B.state->plan;
  const unsigned fill_grid = 4096;
  TG_HIP(hipMemsetAsync(ws.counters, 0, 4 * sizeof(uint32_t), s));  // an earlier call's overflow flag
  for (int32_t c0 = 0; c0 < ns; c0 += S) {
    const int32_t cn = std::min<int32_t>(S, ns - c0);
    TG_HIP(hipMemsetAsync(B.masks, 0, (size_t)n * 4 * sizeof(u64), s));
    TG_HIP(hipMemsetAsync(ws.bits_a, 0, ws.nwords * sizeof(uint32_t), s));
    TG_HIP(hipMemsetAsync(B.state, 0, sizeof(MsState), s));
    hipLaunchKernelGGL(k_bb_fill<float4>, dim3(fill_grid), dim3(BLOCK), 0, s, reinterpret_cast<float4 *>(B.delta),
                       n * S / 4, make_float4(0.f, 0.f, 0.f, 0.f));
    Sources roots;
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
    int32_t L = 0;
    int64_t mu[S];
    for (int64_t &x : mu) x = g.m;
    // the level of the queue at noff: its masks, its edges per source, and
    // the plan on the host
    const auto settle = [&](int64_t noff, u64 *front_new, int32_t level) -> int {
      // few blocks: each ends with an atomic per source
      hipLaunchKernelGGL(k_bb_finalize, dim3((unsigned)std::min<int64_t>(nblk(n), 512)), dim3(BLOCK), 0, s, ws.plan,
                         B.queue_all + noff, B.qmask + noff, B.visited, front_new, B.next, g.out.off,
                         B.state->mf[level & 1], B.state->mf[(level + 1) & 1]);
      TG_HIP(hipMemcpyAsync(B.h_state, B.state, sizeof(MsState), hipMemcpyDeviceToHost, s));
      TG_HIP(hipStreamSynchronize(s));
      return TG_OK;
    };
    TG_TRY(settle(0, B.front[cur], 0));
    for (;;) {
      if (L > g.n) return set_error(TG_EDEVICE, "bc_batched: more supersteps than vertices");
      const Plan P = B.h_state->plan;
      plans.push_back(P);
      segoff.push_back(off);
      const int64_t noff = off + P.count;
      TG_TRY(B.grow(noff + n, noff, s));
      u64 mf[S] = {}, alive = 0;
      for (int c = 0; c < MF_COPIES; ++c)
        for (int k = 0; k < S; ++k) mf[k] += B.h_state->mf[L & 1][c][k];
      for (int k = 0; k < S; ++k) {
        if (mf[k]) alive |= 1ull << k;
        mu[k] -= (int64_t)mf[k];
      }
      TG_TRY(ms_expand(g, ws, t, P, B.queue_all + off, B.front[cur], B.visited, B.next, alive,
                       ms_pull_slots(mf, mu, alive, t), s));
      TG_TRY(frontier_compact(g, ws, 1, ws.bits_a, nullptr, B.queue_all + noff, nullptr, 0, s));
      TG_TRY(frontier_plan(g, ws, B.queue_all + noff, t, s, false));
      TG_TRY(settle(noff, B.front[cur ^ 1], L + 1));
      TG_HIP(hipGetLastError());
      if (B.h_state->plan.count == 0) break;
      const int tk = ktimer_start(s);
      TG_TRY(launch_rows(B.h_state->plan, B.queue_all + noff, B.qmask + noff, g.in.off, g.in.col, B.front[cur],
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
      hipLaunchKernelGGL(k_bb_score, dim3((unsigned)std::min<int64_t>(nblk(g.n * 16), 16384)), dim3(BLOCK), 0, s,
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
