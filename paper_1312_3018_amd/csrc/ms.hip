// Push and pull expansion of a multi-source frontier (see ms.h).
#include <algorithm>

#include "ms.h"

using namespace tgk;

namespace tg {
namespace {

// Push the slots of `take`: new bits of a neighbour = frontier(v) & ~visited.
// The atomic ORs return nothing and are skipped for bits already there; the
// four edges of a lane have their mask reads in flight together.
__global__ __launch_bounds__(BLOCK) void k_ms_push(const Plan *__restrict__ Pp, const int32_t *__restrict__ queue,
                                                   const int64_t *__restrict__ hubpref,
                                                   const int64_t *__restrict__ off, const int32_t *__restrict__ col,
                                                   const u64 *front, const u64 *visited, u64 *next,
                                                   uint32_t *touched, u64 take, int64_t hub_chunk,
                                                   unsigned long long *work) {
  const Plan &P = load_plan(Pp);
  const int lane = threadIdx.x & 63;
  const int64_t total = P.vb[NBIN];
  for (int64_t vb = blockIdx.x; vb < total; vb += gridDim.x) {
    const Assign a = assign_work(vb, P, queue, nullptr, hubpref, off, hub_chunk);
    const u64 m = a.ok ? front[a.v] & take : 0ull;
    const int64_t st = a.stride;
    for (int64_t e = a.e_begin + a.lane; m != 0 && e < a.e_end; e += 4 * st) {
      int32_t nb[4];
      u64 seen[4], have[4];
      uint32_t word[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) nb[q] = e + q * st < a.e_end ? stream_load(col + e + q * st) : -1;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (nb[q] >= 0) {
          seen[q] = visited[nb[q]];
          have[q] = next[nb[q]];
          word[q] = touched[nb[q] >> 5];
        }
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (nb[q] >= 0) {
          const u64 x = m & ~seen[q];
          const uint32_t bit = 1u << (nb[q] & 31);
          if (x & ~have[q]) atomicOr(next + nb[q], x);
          if (x && !(word[q] & bit)) atomicOr(touched + (nb[q] >> 5), bit);
        }
    }
    // (added last: a later read would wait for the additions)
    const bool lead = m != 0 && a.lane == 0;
    const uint32_t k = lead ? (uint32_t)__popcll(m) : 0u;
    const u64 len = lead ? (u64)k * (u64)(a.e_end - a.e_begin) : 0ull;
    const u64 edges = (u64)wave_total((uint32_t)len & 0xFFFFu) + ((u64)wave_total((uint32_t)(len >> 16)) << 16);
    const uint32_t pairs = wave_total(lead && (a.bin != BIN_HUB || a.e_begin == off[a.v]) ? k : 0u);
    if (lane == 0 && edges) {
      stat_add(stat_counter(work, MS_EDGES), edges);
      if (pairs) stat_add(stat_counter(work, MS_PAIRS), (u64)pairs);
    }
  }
}

// The edges looked at and vertices that looked of a block's waves (each
// wave-uniform), to their counters.
__device__ __forceinline__ void publish_pulls(u64 checked, u64 examined, unsigned long long *work) {
  __shared__ u64 part[BLOCK / 64][2];
  if ((threadIdx.x & 63) == 0) {
    part[threadIdx.x >> 6][0] = checked;
    part[threadIdx.x >> 6][1] = examined;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    u64 x = 0;
    for (int k = 0; k < BLOCK / 64; ++k) x += part[k][threadIdx.x];
    if (x) stat_add(stat_counter(work, threadIdx.x == 0 ? MS_CHECKED : MS_EXAMINED), x);
  }
}

// The rows of vertices [0, hubs), HUB_WAVES waves each, one tile of 256 edges
// after another in turn: a slot that is still far from a hub makes all of
// its row be read, 0.8 ms where one wave did it alone.
constexpr int HUB_WAVES = 8;
template <typename OffT>
__global__ __launch_bounds__(BLOCK) void k_ms_pull_hubs(const OffT *__restrict__ ioff,
                                                        const int32_t *__restrict__ icol,
                                                        const u64 *__restrict__ front,
                                                        const u64 *__restrict__ visited, u64 *next, uint32_t *touched,
                                                        u64 take, int64_t hubs, unsigned long long *work) {
  const int lane = threadIdx.x & 63;
  u64 checked = 0, examined = 0;
  const int64_t nw = (int64_t)gridDim.x * (BLOCK / 64);
  for (int64_t t = (int64_t)blockIdx.x * (BLOCK / 64) + (threadIdx.x >> 6); t < hubs * HUB_WAVES; t += nw) {
    const int64_t v = t / HUB_WAVES;
    const u64 w = lane_mask(take & ~visited[v], 0);
    if (!w) continue;
    const int64_t e0 = lane_i64((int64_t)ioff[v], 0), e1 = lane_i64((int64_t)ioff[v + 1], 0);
    const u64 got = pull_tiles(icol, front, e0 + (t % HUB_WAVES) * 256, e1, HUB_WAVES * 256, w, checked);
    examined += t % HUB_WAVES == 0 ? 1 : 0;
    if (got && lane == 0) {
      atomicOr(next + v, got);
      if (touched) atomicOr(touched + (v >> 5), 1u << (v & 31));
    }
  }
  publish_pulls(checked, examined, work);
}

// Pull the slots of `take` for the vertices [hubs, n), a lane each.
template <typename OffT>
__global__ __launch_bounds__(BLOCK) void k_ms_pull(const OffT *__restrict__ ioff, const int32_t *__restrict__ icol,
                                                   const int4 *__restrict__ head, const u64 *__restrict__ front,
                                                   const u64 *__restrict__ visited, u64 *next, uint32_t *touched,
                                                   u64 take, int64_t hubs, int64_t n, unsigned long long *work) {
  const int lane = threadIdx.x & 63;
  u64 checked = 0, examined = 0;
  const int64_t stride = (int64_t)gridDim.x * BLOCK;
  for (int64_t vb = (hubs & ~(int64_t)63) + (int64_t)blockIdx.x * BLOCK; vb < n; vb += stride) {
    const int64_t v = vb + threadIdx.x;
    const u64 want = v >= hubs && v < n ? take & ~visited[v] : 0ull;
    examined += (u64)__popcll(__ballot(want != 0ull));
    const u64 nb = pull_vertices(ioff, icol, head, front, v, want, checked);
    if (nb) next[v] |= nb;
    // a wave covers two whole words that no other wave touches
    const u64 m = __ballot(nb != 0ull);
    if (lane == 0 && (uint32_t)m) touched[v >> 5] |= (uint32_t)m;
    if (lane == 32 && (uint32_t)(m >> 32)) touched[v >> 5] |= (uint32_t)(m >> 32);
  }
  publish_pulls(checked, examined, work);
}

}  // namespace

// How much sooner than the single search (whose switch is bfs_alpha) a slot
// is pulled: pulled slots share one scan that stops early, pushed ones pay an
// atomic per edge and new bit.  On RMAT-20 a pull of nearly all slots takes 35
// us where a push of the few slots that lag behind takes 1.24 ms; 64-source
// betweenness takes 7.4 ms with 1, 6.7 with 4, 5.9-6.4 from 16 to 1024, 64
// searches on a uniform graph of 1,000,003 vertices 2.08, 1.60 and 1.34-1.47.
constexpr int64_t PULL_GAIN = 32;
u64 ms_pull_slots(const u64 *mf, const int64_t *mu, u64 alive, const Tuning &t) {
  if (!t.bfs_do) return 0;
  u64 pulled = 0;
  for (int s = 0; s < kSlots; ++s)
    if (((alive >> s) & 1ull) && (int64_t)mf[s] * PULL_GAIN > std::max<int64_t>(mu[s], 0) / t.bfs_alpha) pulled |= 1ull << s;
  return pulled;
}

int ms_expand(const GpuPart &g, Workspace &ws, const Tuning &t, const Plan &hp, const int32_t *queue,
              const u64 *front, const u64 *visited, u64 *next, u64 alive, u64 pulled, hipStream_t s) {
  const u64 pushed = alive & ~pulled;
  if (pushed && hp.vb[NBIN] > 0)
    hipLaunchKernelGGL(k_ms_push, dim3(launch_grid(hp.vb[NBIN])), dim3(BLOCK), 0, s, ws.plan, queue, ws.hubpref,
                       g.out.off, g.out.col, front, visited, next, ws.bits_a, pushed, t.hub_chunk, ws.work);
  if (pulled) {
    TG_TRY(ms_pull_hubs(g, ws, ws.bits_a, front, visited, next, pulled, s));
    // vertices with in-edges: a symmetric graph ends them at its degree-0 tail
    const int64_t n = g.in_alias ? g.out_bins.bstart[BIN_ZERO] : g.n, hubs = hub_rows(g);
    const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + BLOCK - 1) / BLOCK, 16384));
    const int4 *head = reinterpret_cast<const int4 *>(g.in_head);
    if (g.in_off32)
      hipLaunchKernelGGL(k_ms_pull<int32_t>, dim3(grid), dim3(BLOCK), 0, s, g.in_off32, g.in.col, head, front, visited,
                         next, ws.bits_a, pulled, hubs, n, ws.work);
    else
      hipLaunchKernelGGL(k_ms_pull<int64_t>, dim3(grid), dim3(BLOCK), 0, s, g.in.off, g.in.col, head, front, visited,
                         next, ws.bits_a, pulled, hubs, n, ws.work);
  }
  TG_HIP(hipGetLastError());
  return TG_OK;
}

int64_t hub_rows(const GpuPart &g) { return g.in_alias ? g.out_bins.bstart[BIN_WAVE] : 0; }

int ms_pull_hubs(const GpuPart &g, Workspace &ws, uint32_t *touched, const u64 *front, const u64 *visited, u64 *next,
                 u64 pulled, hipStream_t s) {
  const int64_t hubs = hub_rows(g);
  if (hubs == 0) return TG_OK;
  const unsigned grid = (unsigned)std::min<int64_t>((hubs * HUB_WAVES + 3) / 4, 8192);
  if (g.in_off32)
    hipLaunchKernelGGL(k_ms_pull_hubs<int32_t>, dim3(grid), dim3(BLOCK), 0, s, g.in_off32, g.in.col, front, visited,
                       next, touched, pulled, hubs, ws.work);
  else
    hipLaunchKernelGGL(k_ms_pull_hubs<int64_t>, dim3(grid), dim3(BLOCK), 0, s, g.in.off, g.in.col, front, visited,
                       next, touched, pulled, hubs, ws.work);
  TG_HIP(hipGetLastError());
  return TG_OK;
}

}  // namespace tg
