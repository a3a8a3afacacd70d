// PageRank pull gather (section 7.1, Figure 14) over sliced columns.
//
// Layout.  The rows (destinations) are taken in windows of WIN consecutive
// ids, sorted by length within the window, and cut into slices of 64: a
// wave's lane owns a row, and the slice's edges are stored column by column,
// so that column j of 64 rows is one coalesced 256-byte load.  Sorting keeps
// the padding small (a slice is as long as its longest row) and the rows of
// a slice near each other in the output.  Longer rows are cut into pieces of
// CHUNK words, each a slice of its own whose 64 lanes add up one sum.  A
// column of row ids (the header) goes before each slice, and a bit array
// tells headers from codes: a wave reads its whole share as one stream, two
// groups of columns ahead of the gathers, whatever the lengths of the slices.
// (Sorting rows in windows and storing slices of them by columns is SELL-C-sigma,
// Kreutzer, Hager, Wellein, Fehske and Bishop, SIAM J. Sci. Comput. 36(5), 2014,
// with C = 64 and sigma = WIN; the stream of shares, its headers, the codes and
// the classes below are not part of it.)
// What a lane does per column is one load of the source's code, one gather
// and one or two additions: no row offsets, no staging in LDS, no reduction
// across lanes (the row-block kernel of pr_rows.hip spends 77 vector
// instructions per 64 edges on those; this one 17).
//
// Two modes:
//   classes  The in-edges are split into 8 classes by the 128-byte line of
//            the contribution they gather (line mod 8), and workgroups of XCD
//            k (blockIdx mod 8) walk class k only, so each XCD's L2 and LDS
//            hold an eighth of the contribution vector.  One workgroup per
//            CU keeps the class's hottest contributions in LDS (up to 1022
//            lines), and edges from those are stored two to a word.  A word
//            serves both memories without a branch: a hot word reads the
//            zero before the global vector and a cold one the zero after the
//            table.  Each class leaves a partial sum per row; a combine pass
//            adds the eight and applies the update.  Shares are taken from a
//            counter per class, as columns of hubs and of leaves differ in
//            cost (fixed shares of equal length: waves of 45 to 222 us).
//   whole    One class, no table: on a small graph the contribution vector
//            is in every L2, and loading tables would cost more than the
//            gathers.  A row is finished where it is summed, so that an
//            iteration is one launch.
// Correctness does not depend on the XCD mapping, only the cache behaviour
// does.  Sums run in fp64 in a fixed order, so results are deterministic.
//
// Bound by the gathers that miss LDS (23 M L2 requests per iteration on
// RMAT-22, 128 M edges, where the stream alone takes about 110 us).  Gather of
// an iteration: 433 us in row blocks, 306 us in slices of 32-bit codes whose
// classes lie interleaved in memory (4 of an XCD's 16 L2 channels serve all
// its gathers), 209 us so; the 20-iteration call 9.48 -> 4.77 ms.  R-MAT with
// 30,011 vertices, directed, dangling mass dropped: 19.6 us per iteration in
// four launches, 7.8 us in one (8.9 with the sums of the dangling mass that
// this mode has no use for).
#include <string.h>

#include <algorithm>
#include <vector>

#include "ms.h"

using namespace tgk;

namespace tg {
namespace {

constexpr int NS = 8;      // source classes = XCDs
constexpr int LINE = 32;   // contributions per 128-byte cache line
constexpr int WIN = 512;   // rows sorted together
// Longest row (in words) kept in slices.  Classes, RMAT-22, 20 iterations:
// 64 5.4 ms, 128 4.77, 256 4.76 (a row just past the limit fills half of its
// last column); whole: short slices keep a wave's chain short.
constexpr int LONG_CLS = 128, LONG_WHOLE = 32;
constexpr int CHUNK = 1024;  // words of a piece of a longer row
constexpr int ST = 1024;   // threads per workgroup of the gather
// Columns whose gathers a wave has in flight (codes: twice as many more).
// Classes: 8 0.5 % slower, 24 spills; whole (waves have a few columns only):
// 30,011 vertices, 20 iterations, 16 172 us, 8 166, 4 163.
constexpr int FLY_CLS = 16, FLY_WHOLE = 4;
constexpr int FLYG = 8;    // edges a lane has in flight in a giant
constexpr int SHARES = 4;  // per wave (1: 5.23 ms, 2: 5.00, 4: 4.77, 8: 4.75)
constexpr int PAD = LINE;  // floats before contribution 0 (the last is the zero slot)

// First lane entry of a column group (its header): the lane's row, or NONE;
// LONG_ROW: the 64 lanes' sum is a row's, LONG_PART: a partial's.
constexpr uint32_t NONE = 0xFFFFFFFFu, LONG_ROW = 0x40000000u, LONG_PART = 0x60000000u;
constexpr uint32_t LONG_BITS = 0x60000000u, ID_BITS = 0x1FFFFFFFu;

// A word of class mode: the places of two contributions in the LDS table (15
// bits each, the table's last is a zero), or COLD + the byte offset of one in
// the global vector (whose place 0 is a zero).  Whole mode: the byte offset.
constexpr uint32_t COLD = 0x80000000u;
constexpr int32_t MAX_LINES = 1023;

// Place of source u's contribution.  Classes are stored one after another
// (`stride` floats each): lines 8 apart would share 4 of an XCD's 16 L2
// channels.  stride 0: whole mode, no classes.
__device__ __forceinline__ int64_t place_of(int64_t u, int64_t stride) {
  return stride == 0 ? u : (u >> 5 & (NS - 1)) * stride + (u >> 8 << 5) + (u & 31);
}

// A row summed by a whole block (whole mode): its codes and its length.
struct Giant {
  int64_t e0;
  int32_t len;
  int32_t row;
};

constexpr int64_t GIANT_DEST = (int64_t)1 << 62;

struct WinTotal {  // per class and window
  int32_t slices, cols;  // with the long rows' pieces, and headers
  int32_t rows, slots;   // long rows of several pieces and their pieces (whole mode: giants)
  int64_t edges;         // of the giants
};
struct WinBase {
  int32_t slice, col, row, slot;
  int64_t edge;
};

// ------------------------------------------------------------------- build

// Words per class of every row (one class: the row's length), and in hotw
// those that hold two hot edges (lines below `lines` of each class) each.
template <bool CLS>
__global__ __launch_bounds__(BLOCK) void k_sell_count(const int64_t *__restrict__ off,
                                                      const int32_t *__restrict__ col, int64_t nrows, int32_t lines,
                                                      int32_t *__restrict__ cnt, int32_t *__restrict__ hotw) {
  if (!CLS) {
    const int64_t v = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
    if (v < nrows) cnt[v] = (int32_t)(off[v + 1] - off[v]);
    return;
  }
  const int lane = threadIdx.x & 63;
  const int64_t nw = ((int64_t)gridDim.x * BLOCK) >> 6;
  for (int64_t v = ((int64_t)blockIdx.x * BLOCK + threadIdx.x) >> 6; v < nrows; v += nw) {
    const int64_t e0 = off[v], e1 = off[v + 1];
    int32_t all = 0, hot = 0;  // lane j < 8 keeps the counts of class j
    for (int64_t e = e0; e < e1; e += 64) {
      const int32_t u = e + lane < e1 ? col[e + lane] : 0;
      const int k = e + lane < e1 ? line_class(u) : -1;
      const uint64_t hm = __ballot((u >> 8) < lines);
#pragma unroll
      for (int j = 0; j < NS; ++j) {
        const uint64_t mk = __ballot(k == j);
        if (lane == j) {
          all += __popcll(mk);
          hot += __popcll(mk & hm);
        }
      }
    }
    if (lane < NS) {
      const int32_t hw = (hot + 1) / 2;
      cnt[(int64_t)lane * nrows + v] = hw + all - hot;
      hotw[(int64_t)lane * nrows + v] = hw;
    }
  }
}

// One block per (window, class): sort the window's rows by decreasing length
// (those past `lim` last), note the order in perm[k][w * WIN + i] (-1: none)
// and the window's totals.  In whole mode rows without edges are kept, as
// columnless lanes.
__global__ __launch_bounds__(BLOCK) void k_sell_sort(const int32_t *__restrict__ cnt, int64_t nrows, int64_t nwin,
                                                     int lim, int whole, int32_t *__restrict__ perm,
                                                     WinTotal *__restrict__ tot) {
  __shared__ uint32_t key[WIN];
  __shared__ WinTotal T;
  const int64_t w = blockIdx.x, k = blockIdx.y;
  const int t = threadIdx.x;
  const uint32_t is_long = (uint32_t)lim + 1, none = (uint32_t)lim + 2;
  for (int i = t; i < WIN; i += BLOCK) {
    const int64_t v = w * WIN + i;
    uint32_t rank = none;
    if (v < nrows) {
      const int32_t len = cnt[k * nrows + v];
      rank = len > lim ? is_long : len > 0 || whole ? (uint32_t)(lim - len) : none;
    }
    key[i] = rank * WIN + (uint32_t)i;
  }
  if (t == 0) T = WinTotal{0, 0, 0, 0, 0};
  for (int size = 2; size <= WIN; size <<= 1)
    for (int d = size >> 1; d > 0; d >>= 1) {
      __syncthreads();
      for (int p = t; p < WIN / 2; p += BLOCK) {
        const int i = 2 * p - (p & (d - 1)), j = i + d;
        const uint32_t a = key[i], b = key[j];
        if ((a > b) == ((i & size) == 0)) {
          key[i] = b;
          key[j] = a;
        }
      }
    }
  __syncthreads();
  for (int i = t; i < WIN; i += BLOCK) {
    const uint32_t rank = key[i] / WIN;
    const int32_t v = (int32_t)(w * WIN + (key[i] & (WIN - 1)));
    perm[(k * nwin + w) * WIN + i] = rank == none ? -1 : v;
    if ((i & 63) == 0 && rank <= (uint32_t)lim) {
      atomicAdd(&T.slices, 1);
      atomicAdd(&T.cols, lim - (int32_t)rank + 1);
    }
    if (rank == is_long) {
      const int32_t len = cnt[k * nrows + v], np = (len + CHUNK - 1) / CHUNK;
      if (np > 1) atomicAdd(&T.rows, 1);
      if (np > 1 && whole) {
        atomicAdd(reinterpret_cast<unsigned long long *>(&T.edges), (unsigned long long)len);
      } else {
        if (np > 1) atomicAdd(&T.slots, np);
        atomicAdd(&T.slices, np);
        atomicAdd(&T.cols, (len + 63) / 64 + np);
      }
    }
  }
  __syncthreads();
  if (t == 0) tot[k * nwin + w] = T;
}

struct Placed {
  uint32_t *code;               // 64 per column
  int32_t *ptr;                 // first column of each slice (class k's entries k further on)
  unsigned long long *heads;    // a bit per column: it is a header
  int64_t *dest;                // per class and row, see k_sell_place
  Giant *giants;
  int32_t *lr_slot, *lr_n;      // rows of several pieces: first slot, pieces,
  int64_t *lr_pos;              // place of the sum (class mode)
};

// One block per (window, class): the slices' first columns and headers, the
// long rows' pieces, and where each row's edges go: dest >= 0, the first code
// of a slice's lane, codes 64 apart; < 0, -1 - the header of its first piece,
// or -1 - (GIANT_DEST + its first place among the giants' codes).
__global__ __launch_bounds__(BLOCK) void k_sell_place(const int32_t *__restrict__ cnt, int64_t nrows, int64_t nwin,
                                                      const int32_t *__restrict__ perm,
                                                      const WinBase *__restrict__ base,
                                                      const int64_t *__restrict__ class_col, int lim, int whole,
                                                      int64_t n, Placed P) {
  __shared__ int32_t v_of[WIN], len_of[WIN], col0[WIN / 64];
  __shared__ int32_t slice0[WIN], pcol0[WIN], row0[WIN], slot0[WIN];
  __shared__ int64_t edge0[WIN];
  const int64_t w = blockIdx.x, k = blockIdx.y;
  const int t = threadIdx.x;
  const WinBase B = base[k * nwin + w];
  for (int i = t; i < WIN; i += BLOCK) {
    v_of[i] = perm[(k * nwin + w) * WIN + i];
    len_of[i] = v_of[i] >= 0 ? cnt[k * nrows + v_of[i]] : -1;
  }
  __syncthreads();
  if (t == 0) {
    int32_t c = B.col, sc = B.slice;
    for (int s = 0; s < WIN / 64; ++s) {
      col0[s] = c;
      const int32_t len = len_of[s * 64];
      if (len >= 0 && len <= lim) {
        c += len + 1;
        ++sc;
      }
    }
    int32_t r = B.row, sl = B.slot;
    int64_t e = B.edge;
    for (int i = 0; i < WIN; ++i)
      if (len_of[i] > lim) {
        const int32_t np = (len_of[i] + CHUNK - 1) / CHUNK;
        slice0[i] = sc;
        pcol0[i] = c;
        row0[i] = r;
        slot0[i] = sl;
        edge0[i] = e;
        if (np > 1) ++r;
        if (np > 1 && whole) {
          e += len_of[i];
        } else {
          if (np > 1) sl += np;
          sc += np;
          c += (len_of[i] + 63) / 64 + np;
        }
      }
  }
  __syncthreads();
  const int64_t cc = class_col[k];
  const auto header = [&](int64_t slice, int32_t c) {
    P.ptr[slice + k] = c;
    atomicOr(&P.heads[(cc + c) >> 6], 1ull << ((cc + c) & 63));
  };
  for (int i = t; i < WIN; i += BLOCK) {
    const int s = i >> 6;
    const int32_t v = v_of[i], len = len_of[i], first = len_of[s * 64];
    if (first >= 0 && first <= lim) {
      if ((i & 63) == 0) header(B.slice + s, col0[s]);
      P.code[(cc + col0[s]) * 64 + (i & 63)] = len >= 0 && len <= lim ? (uint32_t)v : NONE;
    }
    if (v < 0) continue;
    if (len <= lim) {
      P.dest[k * nrows + v] = (cc + col0[s] + 1) * 64 + (i & 63);
      continue;
    }
    const int32_t np = (len + CHUNK - 1) / CHUNK;
    if (whole && np > 1) {
      P.dest[k * nrows + v] = -1 - (GIANT_DEST + edge0[i]);
      P.giants[row0[i]] = Giant{edge0[i], len, v};
      continue;
    }
    P.dest[k * nrows + v] = -1 - (cc + pcol0[i]) * 64;
    for (int32_t q = 0; q < np; ++q) {
      const int32_t c = pcol0[i] + q * (CHUNK / 64 + 1);
      header(slice0[i] + q, c);
      const uint32_t h = np == 1 ? LONG_ROW | (uint32_t)v : LONG_PART | (uint32_t)(slot0[i] + q);
      for (int l = 0; l < 64; ++l) P.code[(cc + c) * 64 + l] = h;
    }
    if (np > 1) {
      P.lr_slot[row0[i]] = slot0[i];
      P.lr_n[row0[i]] = np;
      P.lr_pos[row0[i]] = k * n + v;
    }
  }
}

__global__ __launch_bounds__(BLOCK) void k_sell_pad(uint32_t *__restrict__ code, int64_t n, uint32_t value) {
  for (int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x; i < n; i += (int64_t)gridDim.x * BLOCK) code[i] = value;
}

// A wave per row writes its edges' codes: in each class the hot ones two to a
// word, the others after them.
template <bool CLS>
__global__ __launch_bounds__(BLOCK) void k_sell_fill(const int64_t *__restrict__ off, const int32_t *__restrict__ col,
                                                     int64_t nrows, const int64_t *__restrict__ dest,
                                                     const int32_t *__restrict__ hotw, int32_t lines, int64_t stride,
                                                     uint32_t *__restrict__ code, uint32_t *__restrict__ gcode) {
  const int lane = threadIdx.x & 63;
  const uint64_t below = (1ull << lane) - 1ull;
  const int64_t nw = ((int64_t)gridDim.x * BLOCK) >> 6;
  for (int64_t v = ((int64_t)blockIdx.x * BLOCK + threadIdx.x) >> 6; v < nrows; v += nw) {
    const int64_t e0 = off[v], e1 = off[v + 1];
    // lane j: where class j's words of the row are, its next hot and cold edge
    const bool mine = lane < (CLS ? NS : 1) && e1 > e0;
    const int64_t d0 = mine ? dest[(int64_t)lane * nrows + v] : 0;
    int64_t hot_done = 0, cold_done = CLS && mine ? hotw[(int64_t)lane * nrows + v] : 0;
    for (int64_t e = e0; e < e1; e += 64) {
      const bool live = e + lane < e1;
      const int32_t u = live ? col[e + lane] : 0;
      const int k = !live ? -1 : CLS ? line_class(u) : 0;
      const bool hot = CLS && (u >> 8) < lines;
      const uint64_t hm = __ballot(hot);
      int64_t base = 0, idx = 0;
#pragma unroll
      for (int j = 0; j < (CLS ? NS : 1); ++j) {
        const uint64_t mk = __ballot(k == j);
        const int64_t dj = __shfl((long long)d0, j, 64), hj = __shfl((long long)hot_done, j, 64),
                      cj = __shfl((long long)cold_done, j, 64);
        if (k == j) {
          base = dj;
          idx = hot ? hj + __popcll(mk & hm & below) : cj + __popcll(mk & ~hm & below);
        }
        if (lane == j) {
          hot_done += __popcll(mk & hm);
          cold_done += __popcll(mk & ~hm);
        }
      }
      if (!live) continue;
      const int64_t word = hot ? idx >> 1 : idx, x = -1 - base;
      uint32_t *to = base >= 0      ? code + base + word * 64
                     : x < GIANT_DEST ? code + x + 64 + word / CHUNK * (CHUNK + 64) + word % CHUNK
                                      : gcode + (x - GIANT_DEST) + word;
      if (hot) reinterpret_cast<uint16_t *>(to)[idx & 1] = (uint16_t)(((u >> 8) << 5) | (u & 31));
      else *to = (CLS ? COLD : 0u) + 4u * (uint32_t)(place_of(u, stride) + 1);
    }
  }
}

struct ClassDims {
  int32_t slice0[NS], slices[NS], col0[NS], cols[NS];
};

// start[k * (shares + 1) + w]: the first column of share w of class k.
__global__ __launch_bounds__(BLOCK) void k_sell_shares(int32_t *__restrict__ ptr, ClassDims D, int32_t shares,
                                                       int32_t *__restrict__ start) {
  const int k = blockIdx.y;
  const int32_t w = (int32_t)blockIdx.x * BLOCK + threadIdx.x;
  if (w > shares) return;
  const int32_t *p = ptr + D.slice0[k] + k;
  const int32_t want = (int32_t)((int64_t)D.cols[k] * w / shares);
  int32_t lo = 0, hi = D.slices[k];
  while (lo < hi) {
    const int32_t mid = (lo + hi) >> 1;
    if (p[mid] < want) lo = mid + 1;
    else hi = mid;
  }
  start[k * (shares + 1) + w] = D.col0[k] + (lo == D.slices[k] ? D.cols[k] : p[lo]);
}

// ------------------------------------------------------------------ gather

struct SellArgs {
  const uint32_t *code;
  const unsigned long long *heads;
  const int32_t *start;
  int32_t waves, shares;                    // of a class
  int32_t table;                            // floats in the LDS table (whole lines)
  const float *c_in;                        // place 0 of the contributions
  int64_t stride;                           // see place_of
  int64_t n;
  float *ps;
  int32_t *taken;                           // per class (a line apart): shares taken after the first ones
  double *chunk_part;
  // whole mode
  const Giant *giants;  // rows of more than CHUNK edges, a block each
  const uint32_t *gcode;
  int32_t ngiants;
  double base, d, inv_n;
  int32_t drop, last, np_in;
  const double *dang_in;  // np_in partials of the dangling mass
  double *dang_out;       // one per block
  const int32_t *od;
  float *c_out;
  const int32_t *g_of_l;
  float *rank_out;
};

// The one or two contributions of a word (x[1] is 0 where it is one).
template <bool CLS>
__device__ __forceinline__ void gather(const float *table, const char *glob, uint32_t word, uint32_t zero,
                                       float (&x)[CLS ? 2 : 1]) {
  if (CLS) {
    // either the table's two or the global one are zeros
    const uint32_t hot = word < COLD ? word : zero, cold = __builtin_elementwise_sub_sat(word, COLD);
    x[0] = table[hot & 0x7FFFu] + *reinterpret_cast<const float *>(glob + cold);
    x[CLS ? 1 : 0] = table[hot >> 16];
  } else {
    x[0] = *reinterpret_cast<const float *>(glob + word);
  }
}

// Keeps the compiler from moving LDS accesses across this point (a wave's own
// are served in order).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ uint64_t readlane64(unsigned long long v, int l) {
  return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l) |
         (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), l) << 32;
}

template <bool CLS>
__global__ __launch_bounds__(ST) void k_pr_sell(const SellArgs A) {
  extern __shared__ float lds[];  // class mode: a window of sums per wave, then the table
  constexpr int FLY = CLS ? FLY_CLS : FLY_WHOLE;
  __shared__ double red[ST / 64];
  const int t = threadIdx.x, lane = t & 63;
  const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
  const int k = CLS ? (int)(blockIdx.x & (NS - 1)) : 0;
  // (a workgroup's waves take shares far apart)
  const int w = CLS ? wv * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3) : (int)blockIdx.x * (ST / 64) + wv;
  float *win = lds + wv * WIN, *table = lds + (ST / 64) * WIN;
  const uint32_t zero = (uint32_t)A.table * 0x10001u;  // the word without contributions
  const char *glob = reinterpret_cast<const char *>(A.c_in - 1);
  if (CLS) {
    const float4 *src = reinterpret_cast<const float4 *>(A.c_in + k * A.stride);
    float4 *dst = reinterpret_cast<float4 *>(table);
    for (int32_t i = t; i < A.table / 4; i += ST) dst[i] = src[i];
    if (t == 0) table[A.table] = 0.0f;
    for (int i = lane; i < WIN; i += 64) win[i] = __uint_as_float(NONE);
    __syncthreads();
  }
  double add = A.base, dang = 0.0;
  // the dangling mass of the last iteration, summed by every wave alike; not
  // before its first columns are on their way
  bool have = CLS || A.drop;
  const auto dangling = [&]() {
    if (have) return;
    have = true;
    double D = 0.0;
    for (int i = lane; i < A.np_in; i += 64) D += A.dang_in[i];
    add = A.base + A.d * wave_sum(D) * A.inv_n;
  };
  // the sum s of row v, of out-degree od, is known
  const auto finish = [&](int32_t v, double s, int32_t od) {
    if (CLS) {
      A.ps[(int64_t)k * A.n + v] = (float)s;
    } else {
      const double r = add + A.d * s;
      if (A.last) A.rank_out[A.g_of_l[v]] = (float)r;
      else if (od > 0) A.c_out[v] = (float)(r / (double)od);
      if (od == 0) dang += r;
    }
  };
  if (!CLS) {
    for (int32_t i = blockIdx.x; i < A.ngiants; i += gridDim.x) {
      const Giant G = A.giants[i];
      dangling();
      double s = 0.0;
      for (int32_t e = t; e < G.len; e += FLYG * ST) {
        uint32_t c[FLYG];
#pragma unroll
        for (int q = 0; q < FLYG; ++q) c[q] = e + q * ST < G.len ? A.gcode[G.e0 + e + q * ST] : 0u;
#pragma unroll
        for (int q = 0; q < FLYG; ++q) {
          float x[CLS ? 2 : 1];
          gather<CLS>(table, glob, c[q], zero, x);
          s += (double)x[0];
        }
      }
      s = wave_sum(s);
      __syncthreads();
      if (lane == 0) red[wv] = s;
      __syncthreads();
      if (t == 0) {
        for (int q = 1; q < ST / 64; ++q) s += red[q];
        finish(G.row, s, A.od[G.row]);
      }
    }
  }
  // this wave's columns [j, j_end), one stream: the codes are read two groups
  // of columns ahead of their gathers, the header bits 62 words at a time
  for (int32_t sh = w, got = 0; sh < A.shares;
       sh = CLS ? __builtin_amdgcn_readfirstlane(got) + A.waves : A.shares) {
    int32_t j = A.start[k * (A.shares + 1) + sh];
    const int32_t j_end = A.start[k * (A.shares + 1) + sh + 1];
    if (CLS && lane == 0) got = atomicAdd(A.taken + k * LINE, 1);
    if (j >= j_end) continue;
    const uint32_t *code = A.code + lane;
    int32_t hbase = j >> 6;
    unsigned long long hv = A.heads[hbase + lane];
    uint32_t c0[FLY], c1[FLY], c2[FLY];
    const auto load = [&](int32_t at, uint32_t (&cc)[FLY]) {
#pragma unroll
      for (int q = 0; q < FLY; ++q) cc[q] = at + q < j_end ? stream_load(code + (int64_t)(at + q) * 64) : zero;
    };
    load(j, c0);
    load(j + FLY, c1);
    dangling();
    uint32_t row = NONE;
    int32_t od = 0;
    double acc = 0.0;
    // class mode: the sums of a window's rows, which come in the order of their
    // lengths, are gathered in LDS and stored together (NONE: not this wave's)
    uint32_t win_at = NONE;
    const auto store_window = [&]() {
      if (win_at == NONE) return;
      float *to = A.ps + (int64_t)k * A.n + (int64_t)win_at * WIN + lane;
      wave_lds_sync();
#pragma unroll
      for (int i = 0; i < WIN; i += 64) {
        const float x = win[i + lane];
        if (__float_as_uint(x) != NONE) to[i] = x;
        win[i + lane] = __uint_as_float(NONE);
      }
      wave_lds_sync();
    };
    const auto flush = [&]() {
      const uint32_t kind = (uint32_t)__builtin_amdgcn_readfirstlane((int)row);
      if (kind != NONE && (kind & LONG_BITS) != 0) {
        const double s = wave_sum(acc);
        if (lane == 0) {
          if ((kind & LONG_BITS) == LONG_PART) A.chunk_part[kind & ID_BITS] = s;
          else finish((int32_t)(kind & ID_BITS), s, od);
        }
      } else if (CLS) {
        if (kind != NONE && kind / WIN != win_at) {
          store_window();
          win_at = kind / WIN;
        }
        if (row != NONE) win[row % WIN] = (float)acc;
      } else if (row != NONE) {
        finish((int32_t)row, acc, od);
      }
    };
    for (; j < j_end; j += FLY) {
      if ((j >> 6) + 1 - hbase >= 64) {
        hbase = j >> 6;
        hv = A.heads[hbase + lane];
      }
      const int hw = (j >> 6) - hbase, hs = j & 63;
      const uint64_t lo = readlane64(hv, hw), hi = readlane64(hv, hw + 1);
      uint32_t heads = (uint32_t)((lo >> hs) | (hi << 1 << (63 - hs)));
      if (j_end - j < FLY) heads &= (1u << (j_end - j)) - 1u;
      float x[FLY][CLS ? 2 : 1];
#pragma unroll
      for (int q = 0; q < FLY; ++q) gather<CLS>(table, glob, heads >> q & 1u ? zero : c0[q], zero, x[q]);
      load(j + 2 * FLY, c2);
#pragma unroll
      for (int q = 0; q < FLY; ++q) {
        if (heads >> q & 1u) {
          flush();
          acc = 0.0;
          row = c0[q];
          if (!CLS) od = row != NONE ? A.od[row & ID_BITS] : 0;
        } else {
          acc += (double)x[q][0];
          if (CLS) acc += (double)x[q][CLS ? 1 : 0];
        }
      }
#pragma unroll
      for (int q = 0; q < FLY; ++q) {
        c0[q] = c1[q];
        c1[q] = c2[q];
      }
    }
    flush();
    if (CLS) store_window();
  }
  if (CLS || A.drop) return;
  // dangling partial of this workgroup
  dang = wave_sum(dang);
  __syncthreads();
  if (lane == 0) red[wv] = dang;
  __syncthreads();
  if (t < ST / 64) {
    const double s = group_sum(red[t], ST / 64);
    if (t == 0) A.dang_out[blockIdx.x] = s;
  }
}

// Long rows of several pieces: one wave per row adds the pieces' sums.
__global__ __launch_bounds__(BLOCK) void k_pr_sell_long(const int32_t *__restrict__ slot, const int32_t *__restrict__ np,
                                                        const int64_t *__restrict__ pos, int64_t nlr,
                                                        const double *__restrict__ part, float *__restrict__ ps) {
  const int lane = threadIdx.x & 63;
  const int64_t nw = ((int64_t)gridDim.x * BLOCK) >> 6;
  for (int64_t i = ((int64_t)blockIdx.x * BLOCK + threadIdx.x) >> 6; i < nlr; i += nw) {
    double s = 0.0;
    for (int32_t q = lane; q < np[i]; q += 64) s += part[slot[i] + q];
    s = wave_sum(s);
    if (lane == 0) ps[pos[i]] = (float)s;
  }
}

// r(v) = (1-d)/N + d (sum of the 8 partials + D/N); contribution, rank and the
// dangling mass.  Every block adds the last iteration's dangling partials
// itself and leaves its own for the next.
constexpr int CGRID = 1024;
__global__ __launch_bounds__(BLOCK) void k_pr_combine(double base, double d, double inv_n, int drop, int last,
                                                      double iso_count, int64_t n_walk, int64_t n,
                                                      const float *__restrict__ ps, const int32_t *__restrict__ od_of,
                                                      const double *__restrict__ dang_in, int np_in,
                                                      double *__restrict__ dang_out, float *__restrict__ c_out, int64_t stride,
                                                      int32_t *__restrict__ taken,
                                                      const int32_t *__restrict__ g_of_l,
                                                      float *__restrict__ rank_out) {
  if (blockIdx.x == 0 && threadIdx.x < NS) taken[threadIdx.x * LINE] = 0;
  double D = 0.0;
  for (int i = threadIdx.x; i < np_in; i += BLOCK) D += dang_in[i];
  D = block_sum(D);
  const double add = base + d * (drop ? 0.0 : D) * inv_n;
  double dang = 0.0;
  for (int64_t v = (int64_t)blockIdx.x * BLOCK + threadIdx.x; v < n_walk; v += (int64_t)gridDim.x * BLOCK) {
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < NS; ++k) s += (double)__builtin_nontemporal_load(ps + (int64_t)k * n + v);
    const double r = add + d * s;
    const int32_t od = od_of[v];
    if (last) rank_out[g_of_l[v]] = (float)r;
    else if (od > 0) __builtin_nontemporal_store((float)(r / (double)od), c_out + place_of(v, stride));
    if (od == 0) dang += r;
  }
  dang = block_sum(dang);
  // (the isolated tail that is not walked holds its share of `add` each)
  if (threadIdx.x == 0) dang_out[blockIdx.x] = dang + (blockIdx.x == 0 ? iso_count * add : 0.0);
}

// Out-degrees, first contributions 1 / (N od) and the zero slots.
__global__ __launch_bounds__(BLOCK) void k_sell_init(const int64_t *__restrict__ off, int64_t n, double inv_n,
                                                     int64_t stride, int32_t *__restrict__ taken,
                                                      int32_t *__restrict__ od, float *__restrict__ c0,
                                                     float *__restrict__ c1, double *__restrict__ dang, double d0) {
  const int64_t v = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (blockIdx.x == 0 && threadIdx.x < PAD) c0[(int)threadIdx.x - PAD] = c1[(int)threadIdx.x - PAD] = 0.0f;
  if (v == 0) *dang = d0;
  if (taken && v < NS) taken[v * LINE] = 0;
  if (v >= n) return;
  const int64_t x = off[v + 1] - off[v];
  od[v] = (int32_t)x;
  const int64_t at = place_of(v, stride);
  c0[at] = x > 0 ? (float)(inv_n / (double)x) : 0.0f;
  if (x == 0) c1[at] = 0.0f;  // (never written by an iteration)
}

}  // namespace

struct PrSlices {
  DevArena arena;
  bool classes = false;
  int32_t lines = 0, grid = 0;  // what it was built for
  bool built = false;
  int64_t nrows = 0;
  int64_t stride = 0;  // see place_of
  uint32_t *gcode = nullptr;
  Placed at{};
  int32_t *start = nullptr;
  double *chunk_part = nullptr;
  int64_t nlr = 0;
  int32_t waves = 0, shares = 0;
  float *ps = nullptr;
  int32_t *taken = nullptr;
  float *c[2] = {nullptr, nullptr};  // contributions (PAD floats before each)
  int32_t *od = nullptr;
  double *dang[2] = {nullptr, nullptr};
};

void pr_slices_free(GpuPart &g) {
  delete g.slices;
  g.slices = nullptr;
}

namespace {

// Small graphs are walked whole (unless "pr_whole" says otherwise): the
// contribution vector is in every L2 and launches are what counts; past this
// the eight copies of the vector no longer fit the L2s beside the edges.  (us
// per iteration, whole / classes, symmetric R-MAT of 2^12, 2^14, 2^16, 2^18,
// 2^19, 2^20 vertices: 9/18, 11/23, 12/28, 40/46, 68/59, 175/67; directed 2^14,
// 2^16, 2^18: 9/19, 12/21, 24/37; uniform of 2^18 and 2^20, 2 and 8 M edges:
// 17/48, 52/71)
constexpr int64_t WHOLE_MAX_EDGES = (int64_t)12 << 20;

template <typename T>
int push(DevArena &a, T **d, const std::vector<T> &h, hipStream_t s) {
  TG_TRY(dalloc(a, d, std::max<size_t>(h.size(), 1)));
  if (!h.empty()) TG_HIP(hipMemcpyAsync(*d, h.data(), h.size() * sizeof(T), hipMemcpyHostToDevice, s));
  return TG_OK;
}

// Lines of each class in the LDS table: what fits beside the zero slot and
// the block's static arrays, and no more than there are.
int32_t table_lines(const Tuning &t, int64_t n) {
  const int64_t room = rows_lds_limit() / 4 - 64 - (ST / 64) * WIN;
  const int64_t lines = std::min<int64_t>(std::min<int64_t>(t.pr_lds_verts, room) / LINE, MAX_LINES);
  return (int32_t)std::max<int64_t>(0, std::min<int64_t>(lines, (n + (int64_t)LINE * NS - 1) / ((int64_t)LINE * NS)));
}

// Build the slices on the device (once per partition and tuning).
int build_slices(tg_partition *p, hipStream_t s) {
  GpuPart &g = p->gpu;
  const Tuning &t = p->tune;
  const int64_t n = g.n, m = g.in.m;
  const bool cls = t.pr_whole < 0 ? m > WHOLE_MAX_EDGES : t.pr_whole == 0;
  const int32_t lines = cls ? table_lines(t, n) : 0;
  const int32_t grid = (int32_t)(cls ? std::max<int64_t>(t.pr_grid / NS, 1) * NS : t.pr_grid);
  if (g.slices && g.slices->built && g.slices->classes == cls && g.slices->lines == lines && g.slices->grid == grid)
    return TG_OK;
  pr_slices_free(g);
  g.slices = new (std::nothrow) PrSlices();
  if (!g.slices) return set_error(TG_ENOMEM, "pagerank: out of host memory");
  PrSlices &S = *g.slices;
  S.classes = cls;
  S.lines = lines;
  S.grid = grid;
  // rows [0, nrows): with classes a symmetric whole-graph partition leaves
  // out its isolated tail (whose partials stay 0)
  S.nrows = g.in_alias && cls ? g.out_bins.bstart[BIN_ZERO] : n;
  S.stride = cls ? (n + NS * LINE - 1) / (NS * LINE) * LINE : 0;
  const int64_t nrows = S.nrows, nwin = (nrows + WIN - 1) / WIN;
  const int nc = cls ? NS : 1, lim = cls ? LONG_CLS : LONG_WHOLE, whole = cls ? 0 : 1;
  const int64_t nw = nc * nwin;
  DevArena tmp;
  int32_t *cnt = nullptr, *perm = nullptr, *hotw = nullptr;
  WinTotal *dtot = nullptr;
  TG_TRY(dalloc(tmp, &cnt, (size_t)std::max<int64_t>(nc * nrows, 1)));
  TG_TRY(dalloc(tmp, &hotw, (size_t)(cls ? std::max<int64_t>(nc * nrows, 1) : 1)));
  TG_TRY(dalloc(tmp, &perm, (size_t)std::max<int64_t>(nw * WIN, 1)));
  TG_TRY(dalloc(tmp, &dtot, (size_t)std::max<int64_t>(nw, 1)));
  const unsigned wgrid = (unsigned)std::max<int64_t>(1, std::min<int64_t>((nrows * 64 + BLOCK - 1) / BLOCK, 8192));
  const dim3 win((unsigned)nwin, (unsigned)nc);
  std::vector<WinTotal> tot((size_t)nw);
  if (nrows > 0) {
    if (cls)
      hipLaunchKernelGGL(k_sell_count<true>, dim3(wgrid), dim3(BLOCK), 0, s, g.in.off, g.in.col, nrows, lines,
                         cnt, hotw);
    else
      hipLaunchKernelGGL(k_sell_count<false>, dim3((unsigned)((nrows + BLOCK - 1) / BLOCK)), dim3(BLOCK), 0, s, g.in.off,
                         g.in.col, nrows, lines, cnt, hotw);
    hipLaunchKernelGGL(k_sell_sort, win, dim3(BLOCK), 0, s, cnt, nrows, nwin, lim, whole, perm, dtot);
    TG_HIP(hipGetLastError());
    TG_HIP(hipMemcpyAsync(tot.data(), dtot, tot.size() * sizeof(WinTotal), hipMemcpyDeviceToHost, s));
  }
  TG_HIP(hipStreamSynchronize(s));
  std::vector<WinBase> base((size_t)nw);
  std::vector<int64_t> class_col((size_t)nc);
  ClassDims dims;
  memset(&dims, 0, sizeof(dims));
  int64_t slices = 0, lrows = 0, slots = 0, gedges = 0, columns = 0;
  for (int k = 0; k < nc; ++k) {
    const int64_t s0 = slices;
    int64_t cols = 0;
    for (int64_t w = k * nwin; w < (k + 1) * nwin; ++w) {
      const WinTotal &T = tot[(size_t)w];
      base[(size_t)w] = WinBase{(int32_t)slices, (int32_t)cols, (int32_t)lrows, (int32_t)slots, gedges};
      slices += T.slices;
      cols += T.cols;
      lrows += T.rows;
      slots += T.slots;
      gedges += T.edges;
    }
    dims.slice0[k] = (int32_t)s0;
    dims.slices[k] = (int32_t)(slices - s0);
    dims.col0[k] = (int32_t)columns;
    dims.cols[k] = (int32_t)cols;
    class_col[(size_t)k] = columns;
    columns += cols;
    if (columns >= ((int64_t)1 << 31) - 1024 || slots > (int64_t)ID_BITS)
      return set_error(TG_EUNSUPPORTED, "pagerank: too many slices");
  }
  S.nlr = lrows;
  S.waves = (cls ? grid / NS : grid) * (ST / 64);
  // (a share is not worth taking for less than 8 columns)
  S.shares = cls ? (int32_t)std::max<int64_t>(1, std::min<int64_t>((int64_t)S.waves * SHARES, columns / (NS * 8))) : S.waves;
  const size_t nl = (size_t)std::max<int64_t>(lrows, 1);
  const size_t hwords = (size_t)(columns / 64) + 66;
  TG_TRY(dalloc(S.arena, &S.at.code, (size_t)std::max<int64_t>(columns, 1) * 64));
  TG_TRY(dalloc(S.arena, &S.gcode, (size_t)std::max<int64_t>(gedges, 1)));
  TG_TRY(dalloc(S.arena, &S.at.heads, hwords));
  TG_TRY(dalloc(tmp, &S.at.ptr, (size_t)(slices + nc)));
  TG_TRY(dalloc(S.arena, &S.at.giants, whole ? nl : 1));
  TG_TRY(dalloc(S.arena, &S.at.lr_slot, whole ? 1 : nl));
  TG_TRY(dalloc(S.arena, &S.at.lr_n, whole ? 1 : nl));
  TG_TRY(dalloc(S.arena, &S.at.lr_pos, whole ? 1 : nl));
  TG_TRY(dalloc(S.arena, &S.chunk_part, whole ? 1 : (size_t)std::max<int64_t>(slots, 1)));
  TG_TRY(dalloc(S.arena, &S.start, (size_t)nc * (S.shares + 1)));
  TG_TRY(dalloc(tmp, &S.at.dest, (size_t)std::max<int64_t>(nc * nrows, 1)));
  WinBase *dbase = nullptr;
  int64_t *dclass = nullptr;
  TG_TRY(push(tmp, &dbase, base, s));
  TG_TRY(push(tmp, &dclass, class_col, s));
  const uint32_t H = (uint32_t)(lines * LINE);
  if (nrows > 0) {
    TG_HIP(hipMemsetAsync(S.at.heads, 0, hwords * sizeof(unsigned long long), s));
    hipLaunchKernelGGL(k_sell_pad, dim3(4096), dim3(BLOCK), 0, s, S.at.code, columns * 64, H * 0x10001u);
    hipLaunchKernelGGL(k_sell_place, win, dim3(BLOCK), 0, s, cnt, nrows, nwin, perm, dbase, dclass, lim, whole, n, S.at);
    if (cls)
      hipLaunchKernelGGL(k_sell_fill<true>, dim3(wgrid), dim3(BLOCK), 0, s, g.in.off, g.in.col, nrows, S.at.dest, hotw,
                         lines, S.stride, S.at.code, S.gcode);
    else
      hipLaunchKernelGGL(k_sell_fill<false>, dim3(wgrid), dim3(BLOCK), 0, s, g.in.off, g.in.col, nrows, S.at.dest, hotw,
                         lines, S.stride, S.at.code, S.gcode);
  }
  hipLaunchKernelGGL(k_sell_shares, dim3((unsigned)(S.shares / BLOCK + 1), (unsigned)nc), dim3(BLOCK), 0, s, S.at.ptr,
                     dims, S.shares, S.start);
  TG_HIP(hipGetLastError());
  if (cls) {
    TG_TRY(dalloc(S.arena, &S.taken, NS * LINE));
    TG_TRY(dalloc(S.arena, &S.ps, (size_t)NS * std::max<int64_t>(n, 1)));
    // rows that are never walked keep partial 0
    TG_HIP(hipMemsetAsync(S.ps, 0, (size_t)NS * std::max<int64_t>(n, 1) * sizeof(float), s));
  }
  for (int b = 0; b < 2; ++b) {
    float *c = nullptr;
    TG_TRY(dalloc(S.arena, &c, (size_t)std::max(n, NS * S.stride) + 2 * PAD));
    S.c[b] = c + PAD;
    TG_TRY(dalloc(S.arena, &S.dang[b], (size_t)std::max(CGRID, grid)));
  }
  TG_TRY(dalloc(S.arena, &S.od, (size_t)std::max<int64_t>(n, 1)));
  TG_HIP(hipStreamSynchronize(s));  // `base` and `tmp` are still read until here
  S.at.dest = nullptr;
  S.at.ptr = nullptr;
  S.built = true;
  return TG_OK;
}

}  // namespace

bool pr_slices_supported(const GpuPart &g) { return g.n > 0 && g.n < ((int64_t)1 << 29) - NS * LINE && g.in.m < ((int64_t)1 << 35); }

int gpu_pagerank_slices(tg_partition *p, double damping, int32_t iters, int mode, float *rank_out, hipStream_t s) {
  GpuPart &g = p->gpu;
  TG_TRY(build_slices(p, s));
  PrSlices &S = *g.slices;
  const double N = (double)g.n_global;
  const int64_t n = g.n;
  // r_0 = 1/N, so c_0(u) = 1/(N outdeg(u)) and D_0 = (#dangling)/N
  hipLaunchKernelGGL(k_sell_init, dim3((unsigned)((n + BLOCK - 1) / BLOCK)), dim3(BLOCK), 0, s, g.out.off, n, 1.0 / N,
                     S.stride, S.taken, S.od, S.c[0], S.c[1], S.dang[0], (double)g.n_dangling / N);
  SellArgs A;
  memset(&A, 0, sizeof(A));
  A.code = S.at.code;
  A.heads = S.at.heads;
  A.start = S.start;
  A.gcode = S.gcode;
  A.waves = S.waves;
  A.shares = S.shares;
  A.table = S.lines * LINE;
  A.n = n;
  A.stride = S.stride;
  A.ps = S.ps;
  A.taken = S.taken;
  A.chunk_part = S.chunk_part;
  A.giants = S.at.giants;
  A.ngiants = S.classes ? 0 : (int32_t)S.nlr;
  A.base = (1.0 - damping) / N;
  A.d = damping;
  A.inv_n = 1.0 / N;
  A.drop = mode == TG_PR_DANGLING_DROP ? 1 : 0;
  A.od = S.od;
  A.g_of_l = g.g_of_l;
  A.rank_out = rank_out;
  int np_in = 1;  // partials of the dangling mass
  for (int32_t k = 0; k < iters; ++k) {
    const bool last = k == iters - 1;
    A.c_in = S.c[k & 1];
    A.c_out = S.c[(k + 1) & 1];
    A.dang_in = S.dang[k & 1];
    A.dang_out = S.dang[(k + 1) & 1];
    A.np_in = np_in;
    A.last = last ? 1 : 0;
    if (!S.classes) {
      const int tk = ktimer_start(s);
      hipLaunchKernelGGL(k_pr_sell<false>, dim3((unsigned)S.grid), dim3(ST), 0, s, A);
      ktimer_stop(tk, s, "pr_gather");
      np_in = S.grid;
      continue;
    }
    const int tk = ktimer_start(s);
    hipLaunchKernelGGL(k_pr_sell<true>, dim3((unsigned)S.grid), dim3(ST), (size_t)(A.table + 1 + (ST / 64) * WIN) * sizeof(float), s, A);
    if (S.nlr > 0)
      hipLaunchKernelGGL(k_pr_sell_long, dim3((unsigned)long_grid(S.nlr)), dim3(BLOCK), 0, s, S.at.lr_slot, S.at.lr_n,
                         S.at.lr_pos, S.nlr, S.chunk_part, S.ps);
    ktimer_stop(tk, s, "pr_slice_gather");
    // isolated vertices (symmetric graphs: the in-degree-0 tail) are walked only
    // when ranks are written; their dangling share is added analytically
    const bool walk_all = !g.in_alias || last;
    const int64_t n_walk = walk_all ? n : S.nrows;
    const int cgrid = (int)std::max<int64_t>(1, std::min<int64_t>((n_walk + BLOCK - 1) / BLOCK, CGRID));
    const int tk2 = ktimer_start(s);
    hipLaunchKernelGGL(k_pr_combine, dim3(cgrid), dim3(BLOCK), 0, s, A.base, A.d, A.inv_n, A.drop, A.last,
                       walk_all ? 0.0 : (double)g.n_isolated, n_walk, n, S.ps, S.od, A.dang_in, np_in, A.dang_out, A.c_out,
                       S.stride, S.taken, g.g_of_l, rank_out);
    ktimer_stop(tk2, s, "pr_combine");
    np_in = cgrid;
  }
  TG_HIP(hipGetLastError());
  return TG_OK;
}

}  // namespace tg
