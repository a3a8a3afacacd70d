// Collect (Appendix 1, the collect callback): move per-vertex state from the
// partition's local id space to the caller's buffer in original id order,
// plus small fill kernels and the BFS parent pass.
#include <algorithm>

#include "tg_internal.h"

using namespace tgk;

namespace {

inline int blocks_for(int64_t n) { return (int)((n + BLOCK - 1) / BLOCK); }

template <typename T>
__global__ __launch_bounds__(BLOCK) void k_fill(T *__restrict__ p, int64_t n, T v) {
  const int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (i < n) p[i] = v;
}

// out[g] = level of local vertex l_of_g[g] if visited, else INF.  Global ids
// that belong to another partition (l < 0) are left untouched.
__global__ __launch_bounds__(BLOCK) void k_collect_levels(const int32_t *__restrict__ l_of_g, int64_t V,
                                                          const uint32_t *__restrict__ visited,
                                                          const int32_t *__restrict__ level,
                                                          int32_t *__restrict__ out) {
  const int64_t gid = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (gid >= V) return;
  const int32_t l = l_of_g[gid];
  if (l < 0) return;
  const bool seen = (visited[l >> 5] >> (l & 31)) & 1u;
  out[gid] = seen ? level[l] : TG_INF;
}

__global__ __launch_bounds__(BLOCK) void k_collect_i32(const int32_t *__restrict__ l_of_g, int64_t V,
                                                       const int32_t *__restrict__ st,
                                                       int32_t *__restrict__ out) {
  const int64_t gid = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (gid >= V) return;
  const int32_t l = l_of_g[gid];
  if (l >= 0) out[gid] = st[l];
}

__global__ __launch_bounds__(BLOCK) void k_collect_f64_f32(const int32_t *__restrict__ l_of_g, int64_t V,
                                                           const double *__restrict__ st,
                                                           float *__restrict__ out) {
  const int64_t gid = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (gid >= V) return;
  const int32_t l = l_of_g[gid];
  if (l >= 0) out[gid] = (float)st[l];
}

// parent[g] of local v: root -> root; unreached -> -1; otherwise the first
// in-neighbour (in local order) whose level is one less.  Deterministic.
//
// Bound by the chain of dependent loads of the longest row, so no lane walks
// a row alone: a wave takes 16 consecutive vertices, four lanes each, which
// look at the first four in-neighbours (rows start with the hubs, where most
// parents are); the rows still open are then walked by the whole wave, 128
// in-neighbours a step, one after another.  A vertex at level 1 has the root
// as its parent and reads no row: those are the rows that hold one match in
// no particular place.  RMAT-14, one root: 434 us with one thread per vertex
// (a hub's row was one lane's serial walk), 13 us so.
__global__ __launch_bounds__(BLOCK) void k_parents(const int32_t *__restrict__ g_of_l, int64_t v0, int64_t n,
                                                   const int64_t *__restrict__ in_off,
                                                   const int32_t *__restrict__ in_col,
                                                   const uint32_t *__restrict__ visited,
                                                   const int32_t *__restrict__ level, int32_t root,
                                                   int32_t *__restrict__ out) {
  const int lane = threadIdx.x & 63, sub = lane & 3;
  // (without bits, unvisited vertices have level TG_INF)
  const auto seen = [&](int64_t u) { return visited ? ((visited[u >> 5] >> (u & 31)) & 1u) != 0u : level[u] != TG_INF; };
  const auto at = [&](int32_t u, int32_t want) { return (!visited || seen(u)) && level[u] == want; };
  const int64_t v = v0 + (((int64_t)blockIdx.x * BLOCK + threadIdx.x) >> 6) * 16 + (lane >> 2);
  int32_t best = -1, want = 0;
  int64_t e0 = 0, e1 = 0;
  bool open = false;
  if (v < n && seen(v)) {
    want = level[v] - 1;
    if (want <= 0) {
      best = root;
    } else {
      e0 = in_off[v];
      e1 = in_off[v + 1];
      open = true;
    }
  }
  int32_t u = -1;
  if (open && e0 + sub < e1) u = in_col[e0 + sub];
  const uint64_t hits = __ballot(u >= 0 && at(u, want));
  const uint32_t mine = (uint32_t)(hits >> (lane & ~3)) & 15u;
  const int32_t first = __shfl(u, (lane & ~3) + (mine ? __ffs(mine) - 1 : 0), 64);
  if (open && mine) {
    best = first;
    open = false;
  }
  for (uint64_t todo = __ballot(open && sub == 0); todo; todo &= todo - 1) {
    const int src = __ffsll((long long)todo) - 1;
    const int64_t a0 = __shfl((long long)e0, src, 64) + 4, a1 = __shfl((long long)e1, src, 64);
    const int32_t w = __shfl(want, src, 64);
    int32_t found = -1;
    for (int64_t e = a0; e < a1; e += 128) {
      const int64_t i0 = e + lane, i1 = i0 + 64;
      const int32_t u0 = i0 < a1 ? in_col[i0] : -1, u1 = i1 < a1 ? in_col[i1] : -1;
      const bool h0 = u0 >= 0 && at(u0, w), h1 = u1 >= 0 && at(u1, w);
      const uint64_t m0 = __ballot(h0), m1 = __ballot(h1);
      if (m0 | m1) {
        found = m0 ? __shfl(u0, __ffsll((long long)m0) - 1, 64) : __shfl(u1, __ffsll((long long)m1) - 1, 64);
        break;
      }
    }
    if ((lane & ~3) == src) best = found;
  }
  if (v < n && sub == 0) out[g_of_l[v]] = best < 0 ? -1 : g_of_l[best];
}

}  // namespace

namespace tg {

int fill_i32(int32_t *p, int64_t n, int32_t v, hipStream_t s) {
  if (n <= 0) return TG_OK;
  hipLaunchKernelGGL(k_fill<int32_t>, dim3(blocks_for(n)), dim3(BLOCK), 0, s, p, n, v);
  TG_HIP(hipGetLastError());
  return TG_OK;
}
int fill_f64(double *p, int64_t n, double v, hipStream_t s) {
  if (n <= 0) return TG_OK;
  hipLaunchKernelGGL(k_fill<double>, dim3(blocks_for(n)), dim3(BLOCK), 0, s, p, n, v);
  TG_HIP(hipGetLastError());
  return TG_OK;
}
int fill_f32(float *p, int64_t n, float v, hipStream_t s) {
  if (n <= 0) return TG_OK;
  hipLaunchKernelGGL(k_fill<float>, dim3(blocks_for(n)), dim3(BLOCK), 0, s, p, n, v);
  TG_HIP(hipGetLastError());
  return TG_OK;
}

int collect_levels(const GpuPart &g, const uint32_t *visited, const int32_t *level, int32_t *out,
                   hipStream_t s) {
  const int64_t V = (int64_t)g.n_global;
  if (V <= 0) return TG_OK;
  hipLaunchKernelGGL(k_collect_levels, dim3(blocks_for(V)), dim3(BLOCK), 0, s, g.l_of_g, V, visited,
                     level, out);
  TG_HIP(hipGetLastError());
  return TG_OK;
}

int collect_i32(const GpuPart &g, const int32_t *state, int32_t *out, hipStream_t s) {
  const int64_t V = (int64_t)g.n_global;
  if (V <= 0) return TG_OK;
  hipLaunchKernelGGL(k_collect_i32, dim3(blocks_for(V)), dim3(BLOCK), 0, s, g.l_of_g, V, state, out);
  TG_HIP(hipGetLastError());
  return TG_OK;
}

int collect_f64_to_f32(const GpuPart &g, const double *state, float *out, hipStream_t s) {
  const int64_t V = (int64_t)g.n_global;
  if (V <= 0) return TG_OK;
  hipLaunchKernelGGL(k_collect_f64_f32, dim3(blocks_for(V)), dim3(BLOCK), 0, s, g.l_of_g, V, state,
                     out);
  TG_HIP(hipGetLastError());
  return TG_OK;
}

int bfs_parents(const GpuPart &g, const uint32_t *visited, const int32_t *level, int32_t root_local,
                int32_t *out, hipStream_t s) {
  if (g.n <= 0) return TG_OK;
  // four threads a vertex would wrap a launch's 32-bit count from 2^30 on
  constexpr int64_t CHUNK = 1 << 22;
  for (int64_t v0 = 0; v0 < g.n; v0 += CHUNK)
    hipLaunchKernelGGL(k_parents, dim3((unsigned)((std::min(g.n - v0, CHUNK) + BLOCK / 4 - 1) / (BLOCK / 4))), dim3(BLOCK),
                       0, s, g.g_of_l, v0, g.n, g.in.off, g.in.col, visited, level, root_local, out);
  TG_HIP(hipGetLastError());
  return TG_OK;
}

}  // namespace tg
