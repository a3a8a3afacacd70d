// SSSP by buckets for several roots at once, driven on the device.
//
// The schedule is gpu_sssp_ring's (sssp.hip; section 7.3, Figure 20, with
// Meyer and Sanders' delta-stepping): a ring of bucket bitmaps, light edges
// relaxed until a bucket is empty, then the heavy edges of its members once,
// pushed or pulled.  There each superstep is five launches and a wait of the
// host per root; with 50 supersteps a root on a large R-MAT graph those, and
// bitmap passes that leave most of the chip idle, cost more than the edges.
// Here up to ROOTS searches share every launch, and a superstep is three:
//   k_bucket_advance  one thread per root chooses its next pass;
//   k_bucket_collect  turns the pass's vertices into queues, one per degree
//                     bin (a bin is a range of ids, so its queue's room is
//                     known and its order does not matter);
//   k_bucket_relax    a fixed grid walks the queues of all roots, root by
//                     root, so that a root's distances stay in the caches.
// The host only launches ahead and looks at the control blocks once per
// chunk of supersteps.  Which bitmaps of the ring may hold marks is noted by
// the relaxations, so that no pass looks for the next bucket.  A mark stands
// for 32 vertices, a line of distances: whether one of them is active is read
// from its distance, and one that is marked already is not written again.
//
// Bound by the reads of the dense passes (about 80 G line requests a second
// reach the L2s, half of them neighbours' distances) and by the atomic
// minima.  RMAT-22, 8 roots: 15.2 ms in four lanes of single searches; shared
// launches 9.3; a wave walking its vertices' edges as one list instead of 1 to
// 64 lanes per vertex 8.3; collecting blocks of 4 waves instead of 16 7.9.
// Marks as bits, bytes per vertex or per word of vertices, and non-temporal
// distance reads (10.3) did not help.
#include <string.h>

#include <algorithm>

#include "tg_internal.h"

using namespace tgk;

namespace tg {
namespace {

constexpr int ROOTS = 8;  // searches in a launch (ROOTS * NBIN queue lengths fit a wave)
constexpr int CT = 256;   // threads of a collecting block
constexpr int CW = 256;   // its words: 64 per wave
constexpr int CHUNK_EDGES = 2048;  // of a hub's row per block
constexpr int MAX_RING = 16;

enum { LIGHT = 0, PUSH = 1, PULL = 2, OVER = 3 };

struct Ctl {
  int32_t phase, bucket;
  int32_t count[NBIN];  // queue lengths (HUB: chunks)
  uint32_t touched;     // ring bitmaps that may hold a mark
  int32_t merge;        // the members join the final set before the pass
  int32_t light, heavy, pulls;  // passes with work so far
  uint32_t ovf;                 // 1: a candidate did not fit; 2: its vertex stayed unreached
  unsigned long long mem_deg, done_deg;  // out-degree sums of the bucket's members, of the final set
};

struct HubChunk {
  int32_t v, c;
};

struct BucketArgs {
  const int64_t *off;
  const uint32_t *cw;
  const int32_t *lcnt, *hcnt;
  Ctl *ctl;
  int32_t *dist, *settled;  // [roots][n]
  uint32_t *ovf;            // [roots][nwords]
  uint8_t *ring;            // [roots][k][nwords]: marks, a byte per 32 vertices
  uint32_t *sets;           // [roots][2][nwords]: the bucket's members, the final set
  int32_t *queue;           // [roots][n]
  HubChunk *hubq;           // [roots][hub_cap]
  unsigned long long *work;
  int64_t n, nwords, m, hub_cap;
  int32_t roots, k, delta;
  int64_t hpull;  // 0: never pull
  BinBounds light, all;
};

__global__ __launch_bounds__(BLOCK) void k_bucket_init(BucketArgs A, const int32_t *__restrict__ roots) {
  const int64_t y = blockIdx.y;
  const int32_t root = roots[y];
  const int64_t marks = A.k * A.nwords;
  for (int64_t v = (int64_t)blockIdx.x * BLOCK + threadIdx.x; v < A.n; v += (int64_t)gridDim.x * BLOCK) {
    A.dist[y * A.n + v] = v == root ? 0 : TG_INF;
    A.settled[y * A.n + v] = TG_INF;
  }
  for (int64_t q = (int64_t)blockIdx.x * BLOCK + threadIdx.x; q < marks; q += (int64_t)gridDim.x * BLOCK) {
    A.ring[y * marks + q] = q == root >> 5 ? 1 : 0;  // bucket 0: distance 0
    if (q < A.nwords) A.ovf[y * A.nwords + q] = A.sets[2 * y * A.nwords + q] = A.sets[(2 * y + 1) * A.nwords + q] = 0u;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    Ctl c;
    memset(&c, 0, sizeof(c));
    c.phase = LIGHT;
    c.touched = 1u;
    A.ctl[y] = c;
  }
}

__global__ void k_bucket_advance(BucketArgs A) {
  const int y = threadIdx.x;
  if (y >= A.roots) return;
  Ctl C = A.ctl[y];
  int32_t phase = C.phase, any = 0;
  if (phase == OVER) return;
  for (int b = 0; b < NBIN; ++b) {
    any |= C.count[b];
    C.count[b] = 0;
  }
  if (any) {
    if (phase == LIGHT) ++C.light;
    else ++C.heavy;
    if (phase == PULL) ++C.pulls;
  }
  C.merge = 0;
  const int cur = C.bucket % A.k;
  bool next = phase != LIGHT;  // the bucket's heavy edges are done
  if (phase == LIGHT && !(C.touched >> cur & 1u)) {
    // settled: its members' heavy edges are relaxed once, pushed from the
    // members or pulled by the vertices not yet final, whichever side holds
    // fewer edges (the pull's weighted by hpull percent)
    const int64_t push = (int64_t)C.mem_deg, pull = A.m - (int64_t)C.done_deg - push;
    phase = pull * 100 < push * A.hpull ? PULL : PUSH;
    next = push == 0;
  }
  if (next) {
    C.done_deg += C.mem_deg;
    C.mem_deg = 0;
    C.merge = 1;
    phase = OVER;
    for (int j = 1; j < A.k; ++j)
      if (C.touched >> ((C.bucket + j) % A.k) & 1u) {
        C.bucket += j;
        phase = LIGHT;
        break;
      }
  }
  if (phase == LIGHT) C.touched &= ~(1u << (C.bucket % A.k));
  C.phase = phase;
  A.ctl[y] = C;
}

constexpr uint32_t NONE = 0xFFFFFFFFu;

__device__ __forceinline__ uint32_t wave_min(uint32_t x) {
  for (int o = 32; o > 0; o >>= 1) x = min(x, (uint32_t)__shfl_xor((int)x, o, 64));
  return x;
}

// The two halves' masks of a wave's word pair p (words in the lanes).
__device__ __forceinline__ unsigned long long pair_of(uint32_t w, int p) {
  return (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)w, p) |
         (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)w, p + 1) << 32;
}

__global__ __launch_bounds__(CT) void k_bucket_collect(const BucketArgs A) {
  constexpr int WAVES = CT / 64, LW = CW / WAVES;  // words per wave
  __shared__ uint32_t wsum[WAVES];
  __shared__ int32_t slot[NBIN];  // queue entry of the block's rank 0, were it in the bin
  __shared__ unsigned long long wdeg[WAVES];
  const int y = blockIdx.y;
  Ctl &C = A.ctl[y];
  const int phase = C.phase, merge = C.merge;
  if (phase == OVER) return;
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int64_t word0 = (int64_t)blockIdx.x * CW + wv * LW, q = word0 + lane;
  const bool own = lane < LW && q < A.nwords;
  uint8_t *mark = A.ring + (y * A.k + C.bucket % A.k) * A.nwords + q;
  uint32_t *members = A.sets + 2 * y * A.nwords, *done = members + A.nwords;
  const int32_t *dist = A.dist + y * A.n;
  int32_t *settled = A.settled + y * A.n;
  const BinBounds &bb = phase == LIGHT ? A.light : A.all;
  const int32_t *len = phase == LIGHT ? A.lcnt : A.hcnt;
  uint32_t w = 0, mem = 0;
  if (own) {
    const int64_t lo = q * 32, end = phase == LIGHT ? A.n : A.all.bstart[BIN_ZERO];
    const uint32_t valid = lo + 32 <= end ? 0xFFFFFFFFu : lo >= end ? 0u : (1u << (end - lo)) - 1u;
    if (phase == LIGHT) {
      if (*mark) {
        *mark = 0;
        w = valid;
      }
      mem = members[q];
      if (merge && mem) {
        done[q] |= mem;
        members[q] = mem = 0u;
      }
    } else {
      mem = members[q];
      w = mem;
      if (phase == PULL) w = ~(mem | done[q]) & valid;
    }
  }
  if (!__syncthreads_or(w != 0u)) return;
  // what is taken: in a light pass the marked words' vertices whose distance
  // is in the bucket and below the one they last relaxed with; of what is
  // taken the queue gets those with edges
  const int32_t lo = C.bucket * A.delta;
  uint32_t keep = 0, queued = 0;
  unsigned long long deg = 0;  // out-degrees of the new members
  for (unsigned long long nz = __ballot(w != 0u), pairs = (nz | (nz >> 1)) & 0x5555555555555555ull; pairs;) {
    int p[4];
    bool mine[4];
    int32_t d[4], st[4], ln[4], rest[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      p[j] = pairs ? __ffsll((long long)pairs) - 1 : -1;
      pairs &= pairs - 1;
      const int64_t v = (word0 + p[j]) * 32 + lane;
      mine[j] = p[j] >= 0 && (pair_of(w, max(p[j], 0)) >> lane & 1ull) != 0ull;
      if (mine[j] && phase == LIGHT) {
        d[j] = dist[v];
        st[j] = settled[v];
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (phase == LIGHT) mine[j] = mine[j] && d[j] < st[j] && d[j] - lo < A.delta;
      if (!mine[j]) continue;
      const int64_t v = (word0 + p[j]) * 32 + lane;
      ln[j] = len[v];
      if (phase == LIGHT) {
        settled[v] = d[j];  // the distance it relaxes with (at least)
        rest[j] = A.hcnt[v];
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (p[j] < 0) continue;
      if (phase == LIGHT && mine[j] && !(pair_of(mem, p[j]) >> lane & 1ull)) deg += (unsigned long long)(ln[j] + rest[j]);
      const unsigned long long km = __ballot(mine[j]), qm = __ballot(mine[j] && ln[j] > 0);
      if (lane == p[j]) {
        keep = (uint32_t)km;
        queued = (uint32_t)qm;
      } else if (lane == p[j] + 1) {
        keep = (uint32_t)(km >> 32);
        queued = (uint32_t)(qm >> 32);
      }
    }
  }
  if (phase == LIGHT && keep) members[q] = mem | keep;
  // ranks within the block, in the order of ids
  uint32_t inc = (uint32_t)__popc(queued);
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t x = __shfl_up(inc, o, 64);
    if (lane >= o) inc += x;
  }
  deg = wave_sum(deg);
  if (lane == 63) {
    wsum[wv] = inc;
    wdeg[wv] = deg;
  }
  __syncthreads();
  uint32_t before = 0, total = 0;
#pragma unroll
  for (int i = 0; i < WAVES; ++i) {
    if (i < wv) before += wsum[i];
    total += wsum[i];
  }
  const uint32_t excl = before + inc - (uint32_t)__popc(queued);
  if (t == 0) {
    unsigned long long s = 0;
    for (int i = 0; i < WAVES; ++i) s += wdeg[i];
    if (s) atomicAdd(&C.mem_deg, s);
  }
  if (total == 0) return;
  // the block's ranks fall to the bins in turn: bin b's are [from[b], from[b + 1])
  __shared__ uint32_t from[NBIN + 1];
  const int64_t v0 = (int64_t)blockIdx.x * CW * 32, v1 = v0 + (int64_t)CW * 32;
  if (t <= NBIN) {
    const int64_t e = t == NBIN ? A.n : bb.bstart[t];
    if (e <= v0) from[t] = 0;
    else if (e >= v1) from[t] = total;
  }
  if (lane < LW)
    for (int b = 0; b <= NBIN; ++b) {
      const int64_t e = b == NBIN ? A.n : bb.bstart[b];
      if (e > v0 && e < v1 && (e >> 5) == q) from[b] = excl + (uint32_t)__popc(queued & ((1u << (e & 31)) - 1u));
    }
  __syncthreads();
  if (t < NBIN && t != BIN_HUB) {
    const int32_t c = (int32_t)(from[t + 1] - from[t]);
    slot[t] = (int32_t)bb.bstart[t] + (c ? atomicAdd(&C.count[t], c) : 0) - (int32_t)from[t];
  }
  __syncthreads();
  int32_t *queue = A.queue + y * A.n;
  HubChunk *hubq = A.hubq + y * A.hub_cap;
  for (unsigned long long nz = __ballot(queued != 0u), pairs = (nz | (nz >> 1)) & 0x5555555555555555ull; pairs;) {
    const int p = __ffsll((long long)pairs) - 1;
    pairs &= pairs - 1;
    const unsigned long long m = pair_of(queued, p);
    const uint32_t rank =
        (uint32_t)__builtin_amdgcn_readlane((int)excl, p) + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
    if (!(m >> lane & 1ull)) continue;
    const int32_t v = (int32_t)((word0 + p) * 32 + lane);
    int b = 0;
#pragma unroll
    for (int i = 1; i < NBIN; ++i) b += v >= bb.bstart[i] ? 1 : 0;
    if (b == BIN_HUB) {
      const int32_t c = (len[v] + CHUNK_EDGES - 1) / CHUNK_EDGES, at = atomicAdd(&C.count[BIN_HUB], c);
      for (int32_t i = 0; i < c; ++i) hubq[at + i] = HubChunk{v, i};
    } else {
      queue[slot[b] + (int32_t)rank] = v;
    }
  }
}

// Queue entries a wave takes at a time, whose edges it walks as one list (so
// that the chain entry, row, distance is paid once for all of them); rows of
// the BLOCK bin and chunks of hubs take a block each.
__device__ __forceinline__ int entries_per_wave(int b) { return b == BIN_WAVE ? 4 : b == BIN_G16 ? 16 : 64; }
__device__ __forceinline__ int entries_per_block(int b) {
  return b <= BIN_BLOCK ? 1 : entries_per_wave(b) * (BLOCK / 64);
}
constexpr int TILES = 4;  // edges per lane in flight

__global__ __launch_bounds__(BLOCK) void k_bucket_relax(const BucketArgs A) {
  __shared__ int32_t first_vb[64], count_of[64], phase_of[ROOTS];
  __shared__ uint32_t touched[ROOTS], best[BLOCK / 64][64];
  const int t = threadIdx.x, wl = t & 63, wv = t >> 6;
  int32_t vbs = 0;  // lane i: virtual blocks before (root, bin) i, bins from hubs to leaves
  {
    const int r = wl / NBIN, b = wl % NBIN;
    int32_t mine = 0, count = 0;
    if (r < A.roots && b != BIN_ZERO && A.ctl[r].phase != OVER) {
      const int vpb = entries_per_block(b);
      count = A.ctl[r].count[b];
      mine = (count + vpb - 1) / vpb;
    }
    int32_t inc = mine;
    for (int o = 1; o < 64; o <<= 1) {
      const int32_t x = __shfl_up(inc, o, 64);
      if (wl >= o) inc += x;
    }
    vbs = inc - mine;
    if (t < 64) {
      first_vb[t] = vbs;
      count_of[t] = count;
    }
  }
  const int32_t total = __builtin_amdgcn_readlane(vbs, 63);  // (entry 63 is empty)
  if ((int32_t)blockIdx.x >= total) return;
  if (t < A.roots) {
    phase_of[t] = A.ctl[t].phase;
    touched[t] = 0u;
  }
  __syncthreads();
  unsigned long long n_edges = 0, n_verts = 0, n_pulled = 0, n_pullv = 0;
  for (int32_t vb = blockIdx.x; vb < total; vb += gridDim.x) {
    const int i = 63 - __clzll((long long)__ballot(vbs <= vb));  // the last entry that starts at or before vb
    const int r = i / NBIN, b = i - r * NBIN;
    const int32_t local = vb - first_vb[i];
    const int phase = phase_of[r];
    const BinBounds &bb = phase == LIGHT ? A.light : A.all;
    int32_t *dist = A.dist + (int64_t)r * A.n;
    uint8_t *ring = A.ring + (int64_t)r * A.k * A.nwords;
    // an improved vertex's word is marked in its bucket (a mark is read
    // before it is written: the memory takes as long over a byte as over an
    // atomic, and most words are marked by many)
    const auto mark = [&](int32_t v, int32_t d) {
      const int slot = (d / A.delta) % A.k;
      atomicMin(dist + v, d);  // no return value: nothing waits on it
      uint8_t *at = ring + (int64_t)slot * A.nwords + (v >> 5);
      if (!*at) *at = 1;
      if (!(touched[r] >> slot & 1u)) atomicOr(&touched[r], 1u << slot);
    };
    // a candidate that does not fit cannot improve a finite distance; it
    // matters only if v stays unreached
    const auto overflow = [&](int32_t v) {
      atomicOr(A.ovf + (int64_t)r * A.nwords + (v >> 5), 1u << (v & 31));
      A.ctl[r].ovf = 1u;
    };
    const auto relax = [&](int32_t dv, uint32_t x, int32_t cur) {
      const int64_t nd = (int64_t)dv + (int64_t)(x >> 24);
      const int32_t u = (int32_t)(x & 0xFFFFFFu);
      if (nd < (int64_t)cur) mark(u, (int32_t)nd);
      else if (nd >= (int64_t)TG_INF && cur == TG_INF) overflow(u);
    };
    // pulled (symmetric graphs: out-edges are in-edges): the least candidate
    // over the heavy edges from members; final vertices could not gain
    const uint32_t *members = A.sets + 2 * (int64_t)r * A.nwords;
    const auto lower = [&](int32_t v, uint32_t cand) {
      if (cand == NONE) return;
      const int32_t cur = dist[v];
      if (cand < (uint32_t)cur) mark(v, (int32_t)cand);
      else if (cand >= (uint32_t)TG_INF && cur == TG_INF) overflow(v);
    };
    if (b <= BIN_BLOCK) {
      HubChunk h{0, 0};
      if (b == BIN_HUB) h = A.hubq[(int64_t)r * A.hub_cap + local];
      else h.v = A.queue[(int64_t)r * A.n + bb.bstart[b] + local];
      const int64_t o = A.off[h.v], l = o + A.lcnt[h.v];
      const int64_t e0 = (phase == LIGHT ? o : l) + (int64_t)h.c * CHUNK_EDGES;
      int64_t end = phase == LIGHT ? l : A.off[h.v + 1];
      if (b == BIN_HUB) end = min(e0 + CHUNK_EDGES, end);
      if (t == 0) {
        const unsigned long long ne = (unsigned long long)(end - e0), nv = h.c == 0 ? 1 : 0;
        if (phase == PULL) n_pulled += ne, n_pullv += nv;
        else n_edges += ne, n_verts += nv;
      }
      const int32_t dv = dist[h.v];
      uint32_t least = NONE;
      for (int64_t e = e0 + t; e < end; e += TILES * BLOCK) {
        uint32_t x[TILES];
        int32_t d[TILES];
#pragma unroll
        for (int j = 0; j < TILES; ++j) x[j] = e + j * BLOCK < end ? stream_load(A.cw + e + j * BLOCK) : 0u;
        if (phase == PULL) {
          uint32_t mw[TILES];
#pragma unroll
          for (int j = 0; j < TILES; ++j) mw[j] = e + j * BLOCK < end ? members[(x[j] & 0xFFFFFFu) >> 5] : 0u;
#pragma unroll
          for (int j = 0; j < TILES; ++j) d[j] = mw[j] >> (x[j] & 31u) & 1u ? dist[x[j] & 0xFFFFFFu] : -1;
#pragma unroll
          for (int j = 0; j < TILES; ++j)
            if (d[j] >= 0) least = min(least, (uint32_t)d[j] + (x[j] >> 24));
        } else {
#pragma unroll
          for (int j = 0; j < TILES; ++j) d[j] = e + j * BLOCK < end ? dist[x[j] & 0xFFFFFFu] : -1;
#pragma unroll
          for (int j = 0; j < TILES; ++j)
            if (d[j] >= 0) relax(dv, x[j], d[j]);
        }
      }
      if (phase == PULL && (least = wave_min(least), wl == 0)) lower(h.v, least);
      continue;
    }
    // a wave's entries
    const int per = entries_per_wave(b), at0 = (local * (BLOCK / 64) + wv) * per;
    const int k = min(per, count_of[i] - at0);
    if (k <= 0) continue;
    int32_t v = 0, dv = 0, len = 0;
    int64_t e0 = 0;
    if (wl < k) {
      v = A.queue[(int64_t)r * A.n + bb.bstart[b] + at0 + wl];
      const int64_t o = A.off[v], l = o + A.lcnt[v];
      e0 = phase == LIGHT ? o : l;
      len = (int32_t)((phase == LIGHT ? l : A.off[v + 1]) - e0);  // (below the BLOCK bin's rows)
      dv = dist[v];
    }
    int32_t inc = len;
    for (int o = 1; o < 64; o <<= 1) {
      const int32_t x = __shfl_up(inc, o, 64);
      if (wl >= o) inc += x;
    }
    const int32_t total_e = __builtin_amdgcn_readlane(inc, 63);
    const int32_t start = wl < k ? inc - len : INT32_MAX;
    e0 -= inc - len;  // edge p of the list is e0(owner) + p
    if (wl == 0) {
      if (phase == PULL) n_pulled += (unsigned long long)total_e, n_pullv += (unsigned long long)k;
      else n_edges += (unsigned long long)total_e, n_verts += (unsigned long long)k;
    }
    if (phase == PULL) best[wv][wl] = NONE;
    for (int32_t t0 = 0; t0 < total_e; t0 += 64 * TILES) {
      uint32_t x[TILES];
      int32_t own[TILES], d[TILES];
#pragma unroll
      for (int j = 0; j < TILES; ++j) {
        // owner of position p: entries (none is empty) that start at or before
        // the tile, and those that start within it up to p (each tells its
        // lane; lane 0's word is not looked at and takes the others')
        const int32_t s0 = t0 + 64 * j, p = s0 + wl;
        const bool in = start > s0 && start - s0 < 64;
        const int told = __builtin_amdgcn_ds_permute(in ? 4 * (start - s0) : 0, 1);
        const unsigned long long m = __ballot(told != 0) & ~1ull;
        own[j] = __popcll(__ballot(start <= s0)) - 1 + __popcll(m & ((2ull << wl) - 1ull));
        const int64_t e = __shfl((long long)e0, own[j], 64) + p;
        x[j] = p < total_e ? A.cw[e] : 0u;
      }
      if (phase == PULL) {
        uint32_t mw[TILES];
#pragma unroll
        for (int j = 0; j < TILES; ++j) mw[j] = t0 + 64 * j + wl < total_e ? members[(x[j] & 0xFFFFFFu) >> 5] : 0u;
#pragma unroll
        for (int j = 0; j < TILES; ++j) d[j] = mw[j] >> (x[j] & 31u) & 1u ? dist[x[j] & 0xFFFFFFu] : -1;
#pragma unroll
        for (int j = 0; j < TILES; ++j)
          if (d[j] >= 0) atomicMin(&best[wv][own[j]], (uint32_t)d[j] + (x[j] >> 24));
      } else {
#pragma unroll
        for (int j = 0; j < TILES; ++j) d[j] = t0 + 64 * j + wl < total_e ? dist[x[j] & 0xFFFFFFu] : -1;
#pragma unroll
        for (int j = 0; j < TILES; ++j) {
          const int32_t from = __shfl(dv, own[j], 64);
          if (d[j] >= 0) relax(from, x[j], d[j]);
        }
      }
    }
    if (phase == PULL && wl < k) lower(v, best[wv][wl]);  // (a wave's LDS accesses are in order)
  }
  __syncthreads();
  if (t < A.roots && (touched[t] & ~A.ctl[t].touched)) atomicOr(&A.ctl[t].touched, touched[t]);
  n_edges = block_sum(n_edges);
  n_verts = block_sum(n_verts);
  n_pulled = block_sum(n_pulled);
  n_pullv = block_sum(n_pullv);
  if (t == 0) {
    if (n_edges + n_verts) {
      stat_add(stat_counter(A.work, 0), n_edges);
      stat_add(stat_counter(A.work, 1), n_verts);
    }
    if (n_pulled + n_pullv) {
      stat_add(stat_counter(A.work, 2), n_pulled);
      stat_add(stat_counter(A.work, 3), n_pullv);
    }
  }
}

__global__ __launch_bounds__(BLOCK) void k_bucket_verdict(BucketArgs A) {
  const int64_t y = blockIdx.y, v = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (v < A.n && A.ctl[y].ovf && ((A.ovf[y * A.nwords + (v >> 5)] >> (v & 31)) & 1u) && A.dist[y * A.n + v] == TG_INF)
    A.ctl[y].ovf = 2u;
}

__global__ __launch_bounds__(BLOCK) void k_bucket_output(const int32_t *__restrict__ l_of_g,
                                                         const int32_t *__restrict__ dist, int64_t n, int64_t V,
                                                         int32_t *__restrict__ out) {
  const int64_t y = blockIdx.y, gid = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (gid < V) out[y * V + gid] = dist[y * n + l_of_g[gid]];
}

}  // namespace

// Scratch (lazy, per partition): the rows of as many roots as a call had, at
// most ROOTS.
struct BucketState {
  DevArena arena;
  BucketArgs args;
  int32_t *roots = nullptr;
  Ctl *h_ctl = nullptr;
  int32_t *h_roots = nullptr;
  unsigned long long *h_work = nullptr;
  ~BucketState() {
    if (h_ctl) TG_QUIET(hipHostFree(h_ctl));
    if (h_roots) TG_QUIET(hipHostFree(h_roots));
    if (h_work) TG_QUIET(hipHostFree(h_work));
  }
};

void buckets_free(tg_partition *p) {
  delete p->buckets;
  p->buckets = nullptr;
}

namespace {

int bucket_state(tg_partition *p, int roots, int32_t k, BucketState **out) {
  const GpuPart &g = p->gpu;
  // (a row's chunks: one per CHUNK_EDGES, and one for the rest)
  const int64_t hub_cap =
      g.m / CHUNK_EDGES + std::max(g.out_bins.bstart[BIN_BLOCK], g.light_bins.bstart[BIN_BLOCK]) + 1;
  if (p->buckets && p->buckets->args.roots >= roots && p->buckets->args.k == k && p->buckets->args.hub_cap >= hub_cap) {
    *out = p->buckets;
    return TG_OK;
  }
  buckets_free(p);
  p->buckets = new (std::nothrow) BucketState();
  if (!p->buckets) return set_error(TG_ENOMEM, "out of host memory");
  BucketState &S = *p->buckets;
  BucketArgs &A = S.args;
  memset(&A, 0, sizeof(A));
  A.n = g.n;
  A.m = g.m;
  A.nwords = (g.n + 31) / 32;
  A.k = k;
  A.hub_cap = hub_cap;
  const size_t R = (size_t)roots;
  TG_TRY(dalloc(S.arena, &S.roots, R));
  TG_TRY(dalloc(S.arena, &A.ctl, R));
  TG_TRY(dalloc(S.arena, &A.dist, R * (size_t)g.n));
  TG_TRY(dalloc(S.arena, &A.settled, R * (size_t)g.n));
  TG_TRY(dalloc(S.arena, &A.queue, R * (size_t)g.n));
  TG_TRY(dalloc(S.arena, &A.ovf, R * (size_t)A.nwords));
  TG_TRY(dalloc(S.arena, &A.ring, R * (size_t)(k * A.nwords)));
  TG_TRY(dalloc(S.arena, &A.sets, R * (size_t)(2 * A.nwords)));
  TG_TRY(dalloc(S.arena, &A.hubq, R * (size_t)A.hub_cap));
  TG_TRY(dalloc(S.arena, &A.work, (size_t)4 * STAT_SPAN));
  TG_HIP(hipHostMalloc((void **)&S.h_ctl, R * sizeof(Ctl), hipHostMallocDefault));
  TG_HIP(hipHostMalloc((void **)&S.h_roots, R * sizeof(int32_t), hipHostMallocDefault));
  TG_HIP(hipHostMalloc((void **)&S.h_work, 4 * STAT_SPAN * sizeof(unsigned long long), hipHostMallocDefault));
  A.roots = roots;
  *out = &S;
  return TG_OK;
}

}  // namespace

// Whether the partition's schedule is the one above (sssp_prepare has run).
bool buckets_supported(const tg_partition *p) {
  const GpuPart &g = p->gpu;
  const Tuning &t = p->tune;
  return g.n > 0 && t.sssp_ring && t.sssp_split && t.sssp_packed && g.out.cw && !t.sssp_xcd && t.sssp_pull <= 0 &&
         t.sssp_delta > 0 && t.sssp_delta < 256 && (g.max_w + 1 + t.sssp_delta - 1) / t.sssp_delta + 1 <= MAX_RING;
}

int bucket_sssp(tg_partition *p, const int32_t *roots_local, int32_t nr, int32_t *dist, hipStream_t s, int64_t *rounds,
                int64_t *pulls) {
  GpuPart &g = p->gpu;
  const Tuning &t = p->tune;
  TG_TRY(sssp_prepare(p, s));
  const int32_t k = (int32_t)((g.max_w + 1 + t.sssp_delta - 1) / t.sssp_delta + 1);
  BucketState *S = nullptr;
  TG_TRY(bucket_state(p, std::min<int>(nr, ROOTS), k, &S));
  const int cap = S->args.roots;
  const int64_t V = g.n_global;
  TG_HIP(hipMemsetAsync(S->args.work, 0, 4 * STAT_SPAN * sizeof(unsigned long long), s));
  for (int64_t c0 = 0; c0 < nr; c0 += cap) {
    BucketArgs A = S->args;
    A.off = g.out.off;
    A.cw = g.out.cw;
    A.lcnt = g.lcnt;
    A.hcnt = g.hcnt;
    A.delta = (int32_t)t.sssp_delta;
    A.hpull = g.in_alias ? t.sssp_hpull : 0;
    A.light = g.light_bins;
    A.all = g.out_bins;
    A.roots = (int32_t)std::min<int64_t>(cap, nr - c0);
    const unsigned y = (unsigned)A.roots;
    for (int i = 0; i < A.roots; ++i) S->h_roots[i] = roots_local[c0 + i];
    TG_HIP(hipMemcpyAsync(S->roots, S->h_roots, y * sizeof(int32_t), hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(k_bucket_init, dim3((unsigned)std::min<int64_t>((g.n + BLOCK - 1) / BLOCK, 2048), y), dim3(BLOCK),
                       0, s, A, S->roots);
    const unsigned cgrid = (unsigned)((A.nwords + CW - 1) / CW);
    int64_t steps = 0;
    for (bool over = false; !over;) {
      // a vertex is relaxed again only for a smaller distance
      if (steps > 16 * g.n + 1024)
        return set_error(TG_EDEVICE, "sssp: no convergence after %lld passes", (long long)steps);
      constexpr int STEPS = 8;
      for (int i = 0; i < STEPS; ++i) {
        const int tk = ktimer_start(s);
        hipLaunchKernelGGL(k_bucket_advance, dim3(1), dim3(64), 0, s, A);
        hipLaunchKernelGGL(k_bucket_collect, dim3(cgrid, y), dim3(CT), 0, s, A);
        ktimer_stop(tk, s, "bucket_collect");
        const int tr = ktimer_start(s);
        hipLaunchKernelGGL(k_bucket_relax, dim3((unsigned)t.sssp_grid), dim3(BLOCK), 0, s, A);
        ktimer_stop(tr, s, "bucket_relax");
      }
      TG_HIP(hipGetLastError());
      steps += STEPS;
      TG_HIP(hipMemcpyAsync(S->h_ctl, A.ctl, y * sizeof(Ctl), hipMemcpyDeviceToHost, s));
      TG_HIP(hipStreamSynchronize(s));
      ktimer_flush();
      over = true;
      for (int i = 0; i < A.roots; ++i) over = over && S->h_ctl[i].phase == OVER;
    }
    bool ovf = false;
    for (int i = 0; i < A.roots; ++i) {
      *rounds += S->h_ctl[i].light + S->h_ctl[i].heavy;
      *pulls += S->h_ctl[i].pulls;
      ovf = ovf || S->h_ctl[i].ovf;
    }
    const dim3 vg((unsigned)((g.n + BLOCK - 1) / BLOCK), y);
    if (ovf) {
      hipLaunchKernelGGL(k_bucket_verdict, vg, dim3(BLOCK), 0, s, A);
      TG_HIP(hipGetLastError());
      TG_HIP(hipMemcpyAsync(S->h_ctl, A.ctl, y * sizeof(Ctl), hipMemcpyDeviceToHost, s));
      TG_HIP(hipStreamSynchronize(s));
      for (int i = 0; i < A.roots; ++i)
        if (S->h_ctl[i].ovf == 2u)
          return set_error(TG_ERANGE, "sssp: a shortest-path distance does not fit below INT32_MAX");
    }
    hipLaunchKernelGGL(k_bucket_output, dim3((unsigned)((V + BLOCK - 1) / BLOCK), y), dim3(BLOCK), 0, s, g.l_of_g,
                       A.dist, g.n, V, dist + c0 * V);
    TG_HIP(hipGetLastError());
  }
  TG_HIP(hipMemcpyAsync(S->h_work, S->args.work, 4 * STAT_SPAN * sizeof(unsigned long long), hipMemcpyDeviceToHost, s));
  TG_HIP(hipStreamSynchronize(s));
  const char *names[4] = {"relaxations", "activations", "heavy_pull_edges_checked", "heavy_pull_vertices"};
  for (int c = 0; c < 4; ++c) {
    unsigned long long sum = 0;
    for (int i = 0; i < STAT_SLOTS; ++i) sum += S->h_work[(size_t)c * STAT_SPAN + (size_t)i * STAT_STRIDE];
    stats_add(names[c], (double)sum);
  }
  stats_add("lanes", cap < nr ? cap : nr);
  return TG_OK;
}

}  // namespace tg
