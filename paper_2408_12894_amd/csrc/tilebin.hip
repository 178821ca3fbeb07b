// Binning of the depth-sorted Gaussians into tile lists through supertiles of 8 x 8 tiles.
//
// The list the blend reads holds, per tile, the Gaussians whose footprint reaches it in depth
// order. Instead of emitting one (tile, Gaussian) record per instance and sorting those K
// records by tile, a Gaussian is listed once per supertile it reaches, with a 64-bit mask of
// the supertile's tiles it covers: a pair. Pairs are several times fewer than instances (1.7
// per Gaussian against 9.9 instances at 1080p / 1M, 3.8 against 73 for the finest level at
// 3840x2160), so what is moved per instance is only the final list entry:
//   1. k_pair_hist   per column of 256 depth-sorted Gaussians (more in frames above 4K), its pairs per
//                    supertile
//   2. k_rs_scan     per supertile, the exclusive prefix of those counts over the columns
//   3. k_pair_place  the pairs (Gaussian, mask), grouped by supertile and in depth order
//                    inside it, and the descriptors of their chunks of 256
//   4. k_chunk_count per chunk, the instances of each of the supertile's 64 tiles
//   5. k_chunk_prefix  per supertile, their prefix over its chunks and each tile's total
//   6. k_tile_starts   the tiles' [start, end) in tile order
//   7. k_chunk_expand  the list: each chunk's Gaussians of each tile, written as one run; beside it
//                      the blend's tile order
// Order: workgroups, ranks inside one, chunks and bits inside one are all in depth order, so
// each tile's list is ascending (depth bits, Gaussian index).
//
// Against emitting (tile, Gaussian) records and radix-sorting them by tile, which moved 52 B per
// instance (8 written, per 8-bit pass 4 + 8 read and 8 written, 4 read for the ranges), measured
// over all these stages together: 157.6M instances (2.5M Gaussians at 3840x2160) 3.19 -> 0.48 ms,
// 43.0M (the 5-level stack at 1080p) 0.79 -> 0.13 ms, 8.4M (1M Gaussians at 1080p) 0.19 -> 0.09
// ms; 3,140 instances at 128x128 (launches only) 23 -> 27 us.
#include <algorithm>

#include "blend_common.h"

namespace flod {

constexpr int kPairWaves = kPairBlock / 64;
constexpr int kPairWords = kPairBlock / 32;       // words of a bit per Gaussian of a workgroup
constexpr int kWinPer = kSuperWindow / kPairBlock;   // supertiles of a window per thread
// A column of the pair counts is kPairBlock Gaussians where all supertiles fit one window (frames up to
// 3840x2160). Beyond, where a count per supertile and 256 Gaussians would take as much as 320 bytes per
// Gaussian (16384x16384; 2.3 GB for the two arrays of 4.4M), it is as many times that as there are windows
// (8 bytes per Gaussian again), while there are kColumnsMin columns to fill the device. More
// Gaussians to a column than that leave too few workgroups to a frame of few windows (sixteen times 256 of
// 1M Gaussians: 874 us a frame instead of 740 at 4096x2160, two windows).
constexpr int kMostSupers = kMaxSide / (kTile * kSuper), kMostWindows = kMostSupers * kMostSupers / kSuperWindow;
constexpr int kColumnBlocks = kMostWindows, kColumnsMin = 256;

struct Supers {
  int tiles_x, tiles_y;
  int nx, n;   // supertiles per row, in all
};

// One Gaussian's rows of tiles: its rectangle and, where neither the rectangle nor what the
// preprocess stored says all, the footprint, whose rows come out as the preprocess counted them.
struct PairRows {
  int x0, y0, x1, y1;
  int before;   // the stored spans count from x0 - before (of a banded one, from its supertile - before)
  bool full, banded, boxed, bands;
  Footprint fp;
  __device__ __forceinline__ void load(uint2 r) {
    x0 = (int)(r.x & 0x3FFu);
    y0 = (int)(r.x >> 16);
    x1 = (int)(r.y & 0xFFFFu);
    y1 = (int)((r.y >> 16) & 0xFFFu);
    full = (r.y & kRectFull) != 0u;
    banded = (r.y & kRectBanded) != 0u;
    boxed = !banded && (r.y & kRectBoxed) != 0u;
    bands = banded && (r.y & kRectBoxed) != 0u;
    before = (int)(r.x >> kRectBefore) & 15;
  }
  __device__ __forceinline__ void load_footprint(const BinIn &bin, uint32_t g, int tiles_y) {
    const float4 a = bin.xyab[g];
    footprint(a.x, a.y, a.z, a.w, bin.cop[g].x, support_span(bin.qsup[g]), tiles_y, fp);
  }
  // supertile columns of supertile row sy that the Gaussian is listed in (the preprocess
  // counted the same): the rectangle's, or of a banded one the union of the row spans
  __device__ __forceinline__ void columns(int sy, const BinIn &bin, uint32_t g, int tiles_x, int &c0, int &c1) const {
    c0 = x0 / kSuper;
    c1 = x1 / kSuper;
    if (!banded) return;
    if (bands) {
      const uint32_t byte = reinterpret_cast<const uint8_t *>(bin.spans + g)[sy - y0 / kSuper];
      const int c = x0 / kSuper - before;
      c0 = c + (int)(byte & 15u);
      c1 = c + (int)(byte >> 4);
      return;
    }
    int u0 = 0x7FFFFFFF, u1 = -1;
    for (int ty = max(y0, sy * kSuper); ty <= min(y1, sy * kSuper + kSuper - 1); ++ty) {
      int a, b;
      if (row_span(fp, ty, tiles_x, a, b)) {
        u0 = min(u0, a);
        u1 = max(u1, b);
      }
    }
    c0 = u0 / kSuper;
    c1 = u1 < 0 ? -1 : u1 / kSuper;
  }
};

// ---------------------------------------------------------------------------------------
// Pairs of each column of `per` Gaussians (one workgroup) per supertile: hist[s * stride + column],
// for the per-supertile scan over the columns; all supertiles' counts in LDS (64 KB at most). The
// columns of large footprints listed row by row are read where
// the preprocess stored them: recomputing their rows in FP64, a serial chain of up to 10 us in
// the few waves that have one, took 17 instead of 8 us at 1M Gaussians / 1080p (0.001% of them)
// and 63 instead of 29 at 2.5M / 3840x2160 (0.14%). What remains there is the 4.3M strided
// 4-byte writes; eight blocks per workgroup, writing 32 bytes at a time, gained nothing (29 us;
// 15 instead of 11 at 2.1M / 1280x720).
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(kPairBlock) void k_pair_hist(const uint32_t *__restrict__ ids,
                                                          const uint32_t *__restrict__ counters,
                                                          const uint2 *__restrict__ srect, BinIn bin, Supers su,
                                                          uint32_t *__restrict__ hist, int stride, uint32_t per) {
  extern __shared__ uint32_t s_cnt[];
  const uint32_t n = counters[kCntVisible];
  if (counters[kCntPairs] == 0u) return;   // no pairs, or more than the buffers hold
  const uint32_t nb = (n + per - 1) / per;
  const uint32_t b = xcd_block(blockIdx.x);
  if (b >= nb) return;
  const uint32_t base = b * per, count = min(per, n - base);
  for (int s = threadIdx.x; s < su.n; s += kPairBlock) s_cnt[s] = 0u;
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < count; i += kPairBlock) {
    PairRows r;
    r.load(srect[base + i]);
    uint32_t g = 0u;
    if (r.banded) g = ids[base + i];
    if (r.banded && !r.bands) r.load_footprint(bin, g, su.tiles_y);
    for (int sy = r.y0 / kSuper; sy * kSuper <= r.y1; ++sy) {
      int c0, c1;
      r.columns(sy, bin, g, su.tiles_x, c0, c1);
      for (int c = c0; c <= c1; ++c) atomicAdd(&s_cnt[sy * su.nx + c], 1u);
    }
  }
  __syncthreads();
  for (int s = threadIdx.x; s < su.n; s += kPairBlock) hist[(size_t)s * stride + b] = s_cnt[s];
}

// Row spans of footprints, the rows of a wave's Gaussians dealt to its lanes in order: those whose
// spans the preprocess stored need none, and of the others, few and tall, a wave would repeat the
// FP64 rows as often as the tallest has rows. rows: this lane's count of rows (0: none), incl:
// its inclusive sum over the lanes. The span of a lane's row r goes to spans[incl - rows + r] as
// x0 | x1 << 16, an empty one as 1. Every lane of the wave takes part; spans is the wave's own.
constexpr int kSpanHold = 1024;   // row spans a wave has room for; no footprint has more rows (frames
                                  // are at most 16384 pixels high)

__device__ __forceinline__ int owner_lane(uint32_t incl, uint32_t v) {
  int lo = 0;   // the number of lanes with incl <= v
#pragma unroll
  for (int step = 32; step > 0; step >>= 1) {
    const uint32_t x = __shfl(incl, lo + step - 1, 64);
    if (x <= v) lo += step;
  }
  return lo;
}

__device__ __forceinline__ void wave_row_spans(const Footprint &f, int y0, uint32_t rows, uint32_t incl, int tiles_x,
                                               uint32_t *spans) {
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t total = __shfl(incl, 63, 64);
  const int first = y0 - (int)(incl - rows);   // row v of the wave's is tile row v + first of its owner
  for (uint32_t v0 = 0; v0 < total; v0 += 64) {
    const uint32_t v = min(v0 + lane, total - 1u);
    const int o = owner_lane(incl, v);
    Footprint g;
    g.mx = __shfl(f.mx, o, 64); g.my = __shfl(f.my, o, 64); g.b = __shfl(f.b, o, 64);
    g.qa = __shfl(f.qa, o, 64); g.det = __shfl(f.det, o, 64); g.ia = __shfl(f.ia, o, 64);
    g.hx = __shfl(f.hx, o, 64); g.hy = __shfl(f.hy, o, 64); g.dyr = __shfl(f.dyr, o, 64);
    int a, e;
    const bool ok = row_span(g, (int)v + __shfl(first, o, 64), tiles_x, a, e);
    if (v0 + lane < total) spans[v] = ok ? (uint32_t)a | ((uint32_t)e << 16) : 1u;
  }
}

// Exclusive scan of two values per thread over the workgroup.
__device__ __forceinline__ void block_excl_scan2(uint32_t &a, uint32_t &b, uint32_t &ta, uint32_t &tb) {
  __shared__ uint32_t s_a[kPairWaves], s_b[kPairWaves];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint32_t ia = wave_incl_scan(a), ib = wave_incl_scan(b);
  __syncthreads();
  if (lane == 63) {
    s_a[w] = ia;
    s_b[w] = ib;
  }
  __syncthreads();
  uint32_t ba = 0, bb = 0;
  ta = tb = 0;
#pragma unroll
  for (int k = 0; k < kPairWaves; ++k) {
    const uint32_t xa = s_a[k], xb = s_b[k];
    ba += k < w ? xa : 0u;
    bb += k < w ? xb : 0u;
    ta += xa;
    tb += xb;
  }
  a = ba + ia - a;
  b = bb + ib - b;
}

// Position of the r-th set bit of m (r below its bit count).
__device__ __forceinline__ uint32_t select_bit(unsigned long long m, uint32_t r) {
  uint32_t at = 0u;
#pragma unroll
  for (int step = 32; step > 0; step >>= 1) {
    const uint32_t c = (uint32_t)__popcll(m & ((1ull << step) - 1ull));
    if (r >= c) {
      r -= c;
      m >>= step;
      at += step;
    }
  }
  return at;
}

// ---------------------------------------------------------------------------------------
// The pairs, each at its supertile's start + the earlier columns' pairs there + its rank
// among the column's. Ranks: one bit per (supertile, Gaussian) in LDS, its prefix over the
// words of a supertile, and a bit count inside the word. Rows: read where the preprocess stored
// them (16 bytes for a footprint of up to 16 x 16 tiles), else computed by the wave into LDS
// (wave_row_spans; as many Gaussians at a time as fit, one at least). Masks: per supertile row
// and four supertiles, each tile row's tiles as 32 bits, whose bytes are then the rows of the
// four masks. Also writes the supertiles' (first chunk, chunks), the chunks' descriptors and
// their count.
// Bound by VALU issue (58% of the cycles) and the scattered 12-byte writes. Each thread computing
// its rows in FP64 and assembling each mask bit range by bit range took 73 us at 1M Gaussians /
// 1080p (1% of the footprints beyond 16 x 16 tiles) and 391 us at 2.5M / 3840x2160 (15%); this
// 40 and 178, for 12 bytes fewer written per Gaussian by the preprocess.
//
// MANY (frames of more than kSuperWindow supertiles): a workgroup takes the pairs that a column of
// `per` Gaussians makes in one window of kSuperWindow supertiles (blockIdx.y). It first marks the Gaussians whose
// rectangles meet the window, then takes those 256 at a time, with the rows that lie in the
// window. Every workgroup of 256 Gaussians going through all windows instead repeated the FP64
// rows and the 16 KB of bits for each, mostly for a handful of pairs: 16384x16384 (32 windows)
// 1,770 us with 2k Gaussians and 2,270 with 4.4M small ones, now 58 and 460.
// ---------------------------------------------------------------------------------------
template <bool MANY>
__global__ __launch_bounds__(kPairBlock, 4) void k_pair_place(
    const uint32_t *__restrict__ ids, uint32_t *counters, const uint2 *__restrict__ srect,
    BinIn bin, Supers su, const uint32_t *__restrict__ scan, const uint32_t *__restrict__ tot, int stride, uint32_t per,
    const uint2 *__restrict__ starts, uint32_t *__restrict__ pair_id, unsigned long long *__restrict__ pair_mask,
    uint4 *__restrict__ chunks, uint2 *__restrict__ supers) {
  // word w of a supertile's bits at w ^ bits_at(s), which spreads 64 supertiles over the banks
  __shared__ uint32_t s_bits[kSuperWindow][kPairWords];
  __shared__ union {
    uint8_t b[kPairWords];   // of the earlier words' bits, at most 224
    uint2 v;
  } s_pre[kSuperWindow];
  __shared__ uint32_t s_goff[kSuperWindow];
  __shared__ union {
    uint32_t span[kPairWaves][kSpanHold];
    uint4 chunk[kSuperWindow];   // first pair, pairs, first chunk, chunks
  } s_u;
  constexpr int kMarks = MANY ? kColumnBlocks * kPairWaves : 1;
  __shared__ unsigned long long s_mark[kMarks];   // the column's Gaussians that meet the window
  __shared__ uint32_t s_first[kMarks];            // and those before each word
  uint4 *s_chunk = s_u.chunk;
  const auto bits_at = [](int s) { return (s >> 3) & (kPairWords - 1); };
  const uint32_t n = counters[kCntVisible];
  if (counters[kCntPairs] == 0u) return;
  if (!MANY) per = kPairBlock;
  const uint32_t nb = (n + per - 1) / per;
  const uint32_t b = xcd_block(blockIdx.x);
  if (b >= nb) return;
  const int tid = threadIdx.x;
  const uint32_t base = b * per, count = min(per, n - base);
  const int w0 = MANY ? (int)blockIdx.y * kSuperWindow : 0, w1 = min(su.n, w0 + kSuperWindow);
  const int word = tid >> 5;
  const uint32_t bit = 1u << (tid & 31);
  const uint32_t marks = MANY ? (count + 63u) / 64u : 0u;
  PairRows r;
  uint32_t g = 0u;
  const auto take = [&](uint32_t j) {
    g = ids[j];
    r.load(srect[j]);
    if (r.boxed) {
      // in place of a footprint its spans: byte q of the three words is tile row q of the supertile
      // rows from its first on
      uint4 e = bin.spans[g];
      e = make_uint4(e.x ^ kSpanNone, e.y ^ kSpanNone, e.z ^ kSpanNone, e.w ^ kSpanNone);   // rows beyond it: none
      const int sh = 8 * (r.y0 % kSuper);
      const unsigned long long lo = ((unsigned long long)e.y << 32) | e.x, hi = ((unsigned long long)e.w << 32) | e.z;
      r.fp.qa = __longlong_as_double((long long)(lo << sh));
      r.fp.det = __longlong_as_double((long long)((hi << sh) | (lo >> 1 >> (63 - sh))));
      r.fp.ia = __longlong_as_double((long long)(hi >> 1 >> (63 - sh)));
    } else if (!r.full) {
      r.load_footprint(bin, g, su.tiles_y);
    }
  };
  const auto clear = [&]() {
#pragma unroll
    for (int k = 0; k < kWinPer; ++k)
#pragma unroll
      for (int w = 0; w < kPairWords; ++w) s_bits[tid * kWinPer + k][w] = 0u;
  };
  const auto none = [&]() {
    r.load(make_uint2(0u, 0u));
    r.y1 = -1;
  };
  none();
  if (!MANY && (uint32_t)tid < count) take(base + tid);
  if (MANY) {
    const int r0 = w0 / su.nx, r1 = (w1 - 1) / su.nx;   // the window's supertile rows
#pragma unroll 4
    for (uint32_t i = tid; i < ((count + 63u) & ~63u); i += kPairBlock) {   // whole waves
      const uint2 q = i < count ? srect[base + i] : make_uint2(0u, 0u);
      PairRows t;
      t.load(q);
      const int c0 = t.x0 / kSuper, c1 = t.x1 / kSuper;
      bool hit = false;
      for (int sy = max(t.y0 / kSuper, r0); sy <= min(t.y1 / kSuper, r1); ++sy)
        hit = hit || (sy * su.nx + c1 >= w0 && sy * su.nx + c0 < w1);
      const unsigned long long m = __ballot(hit && i < count);
      if ((tid & 63) == 0) s_mark[i >> 6] = m;
    }
  }
  {
    // thread t takes the window's supertiles kWinPer t .. kWinPer t + kWinPer - 1
    uint32_t t[kWinPer], sp = 0u, sc = 0u;
#pragma unroll
    for (int k = 0; k < kWinPer; ++k) {
      const int s = w0 + tid * kWinPer + k;
      t[k] = s < w1 ? tot[s] : 0u;
      sp += t[k];
      sc += (t[k] + kChunk - 1) / kChunk;
    }
    uint32_t tp, tc;
    block_excl_scan2(sp, sc, tp, tc);
    if (MANY) {
      const uint2 st = starts[blockIdx.y];
      sp += st.x;
      sc += st.y;
    }
#pragma unroll
    for (int k = 0; k < kWinPer; ++k) {
      const int s = tid * kWinPer + k;
      const uint32_t nc = (t[k] + kChunk - 1) / kChunk;
      s_goff[s] = sp + (w0 + s < w1 ? scan[(size_t)(w0 + s) * stride + b] : 0u);
      s_chunk[s] = make_uint4(sp, t[k], sc, nc);
      sp += t[k];
      sc += nc;
    }
    if (!MANY && b == 0u && tid == 0) counters[kCntChunks] = tc;
    clear();
  }
  __syncthreads();
  // the chunks' descriptors: supertile s by column s mod nb
  for (uint32_t s = b + ((uint32_t)w0 > b ? ((uint32_t)w0 - b + nb - 1) / nb * nb : 0u); s < (uint32_t)w1; s += nb) {
    const uint4 c = s_chunk[s - w0];
    if (tid == 0) supers[s] = make_uint2(c.z, c.w);
    for (uint32_t i = tid; i < c.w; i += kPairBlock)
      chunks[c.z + i] = make_uint4(c.x + i * kChunk, min((uint32_t)kChunk, c.y - i * kChunk), s, 0u);
  }
  uint32_t todo = count;   // Gaussians to take: MANY, the marked ones
  if (MANY) {
    uint32_t before = (uint32_t)tid < marks ? (uint32_t)__popcll(s_mark[tid]) : 0u, zero = 0u, zeros;
    block_excl_scan2(before, zero, todo, zeros);
    if ((uint32_t)tid < marks) s_first[tid] = before;
    __syncthreads();
  }
  // 256 Gaussians at a time (all of the column's unless MANY)
  for (uint32_t at = 0u; at < todo; at += kPairBlock) {
    if (MANY) {
      none();
      if (at + tid < todo) {
        uint32_t k = 0u;   // the last word with at most at + tid marks before it
#pragma unroll
        for (uint32_t step = kMarks / 2; step > 0; step >>= 1)
          if (k + step < marks && s_first[k + step] <= at + tid) k += step;
        take(base + 64u * k + select_bit(s_mark[k], at + tid - s_first[k]));
      }
      if (at > 0u) {
        clear();
        __syncthreads();
      }
    }
    // its tile rows in the window's supertile rows
    const int y0 = MANY ? max(r.y0, w0 / su.nx * kSuper) : r.y0;
    const int y1 = MANY ? min(r.y1, (w1 - 1) / su.nx * kSuper + kSuper - 1) : r.y1;
    for (int sy = y0 / kSuper; sy * kSuper <= y1; ++sy) {
      const int first = sy * su.nx;
      int c0, c1;
      r.columns(sy, bin, g, su.tiles_x, c0, c1);
      if (MANY) {
        c0 = max(c0, w0 - first);
        c1 = min(c1, w1 - 1 - first);
      }
      for (int c = c0; c <= c1; ++c) {
        const int s = first + c - w0;
        atomicOr(&s_bits[s][word ^ bits_at(s)], bit);
      }
    }
    __syncthreads();
    uint32_t taken[kWinPer];   // of this thread's supertiles
#pragma unroll
    for (int k = 0; k < kWinPer; ++k) {
      const int s = tid + k * kPairBlock;
      uint32_t acc = 0u, p[2] = {0u, 0u};
#pragma unroll
      for (int w = 0; w < kPairWords; ++w) {
        p[w >> 2] |= acc << (8 * (w & 3));
        acc += (uint32_t)__popc(s_bits[s][w ^ bits_at(s)]);
      }
      s_pre[s].v = make_uint2(p[0], p[1]);
      taken[k] = acc;
    }
    __syncthreads();
    // this wave's Gaussians, those whose rows fit the spans' room at a time
    uint32_t *spans = s_u.span[tid >> 6];
    bool pending = y1 >= y0;
    while (__any(pending)) {
      const uint32_t need = pending && !r.full && !r.boxed ? (uint32_t)(y1 - y0 + 1) : 0u;
      const uint32_t upto = wave_incl_scan(need);   // every lane takes part
      const bool now = pending && upto <= (uint32_t)kSpanHold;
      const uint32_t rows = now ? need : 0u;
      const uint32_t incl = wave_incl_scan(rows);
      wave_row_spans(r.fp, y0, rows, incl, su.tiles_x, spans);
      wave_lds_fence();
      if (now) {
        const uint32_t *mine = spans + (incl - rows);
        for (int sy = y0 / kSuper; sy * kSuper <= y1; ++sy) {
          const int first = sy * su.nx;
          int ra[kSuper], re[kSuper];   // first and last column, first above last for none
          int c0 = r.x0 / kSuper, c1 = r.x1 / kSuper;
          if (r.boxed) {
            const int k = sy - r.y0 / kSuper;
            const double v = k == 0 ? r.fp.qa : k == 1 ? r.fp.det : r.fp.ia;
            const unsigned long long x = (unsigned long long)__double_as_longlong(v) ^ 0x0101010101010101ull;
            const uint32_t xl = (uint32_t)x, xh = (uint32_t)(x >> 32);
#pragma unroll
            for (int q = 0; q < kSuper; ++q) {
              const uint32_t y = q < 4 ? xl : xh;
              ra[q] = r.x0 - r.before + (int)((y >> (8 * (q & 3))) & 15u);
              re[q] = r.x0 - r.before + (int)((y >> (8 * (q & 3) + 4)) & 15u);
            }
          } else {
            int u0 = 0x7FFFFFFF, u1 = -1;
#pragma unroll
            for (int q = 0; q < kSuper; ++q) {
              const int ty = sy * kSuper + q;
              const bool in = ty >= y0 && ty <= y1;
              const uint32_t s = r.full ? (uint32_t)r.x0 | ((uint32_t)r.x1 << 16) : mine[in ? ty - y0 : 0];
              ra[q] = in ? (int)(s & 0xFFFFu) : 1;
              re[q] = in ? (int)(s >> 16) : 0;
              u0 = ra[q] <= re[q] ? min(u0, ra[q]) : u0;
              u1 = ra[q] <= re[q] ? max(u1, re[q]) : u1;
            }
            if (r.banded) {
              c0 = u0 / kSuper;
              c1 = u1 < 0 ? -1 : u1 / kSuper;
            }
          }
          if (MANY) {
            c0 = max(c0, w0 - first);
            c1 = min(c1, w1 - 1 - first);
          }
          for (int g0 = c0; g0 <= c1; g0 += 4) {
            uint32_t bits[kSuper];   // the row's tiles of four supertiles
#pragma unroll
            for (int q = 0; q < kSuper; ++q) {
              const int a = ra[q] - g0 * kSuper, e = re[q] - g0 * kSuper;
              const uint32_t m = (~0u << min(max(a, 0), 31)) & (~0u >> (31 - min(max(e, 0), 31)));
              bits[q] = a <= e && a < 32 && e >= 0 ? m : 0u;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              if (g0 + k > c1) break;
              uint32_t m[2];
#pragma unroll
              for (int h = 0; h < 2; ++h) {
                const uint32_t *q = bits + 4 * h;   // byte k of the four rows
                const uint32_t sel = (uint32_t)((4 + k) << 8 | k);
                const uint32_t lo = __builtin_amdgcn_perm(q[1], q[0], sel), hi = __builtin_amdgcn_perm(q[3], q[2], sel);
                m[h] = __builtin_amdgcn_perm(hi, lo, 0x05040100u);
              }
              const int s = first + g0 + k - w0;
              const uint32_t rank = s_pre[s].b[word] + (uint32_t)__popc(s_bits[s][word ^ bits_at(s)] & (bit - 1u));
              const uint32_t p = s_goff[s] + rank;
              pair_id[p] = g;
              pair_mask[p] = ((unsigned long long)m[1] << 32) | m[0];
            }
          }
        }
        pending = false;
      }
      wave_lds_fence();
    }
    if (!MANY) break;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kWinPer; ++k) s_goff[tid + k * kPairBlock] += taken[k];
  }
}

// MANY: the first pair and the first chunk of each window of supertiles, and the chunks' count.
__global__ __launch_bounds__(kSuperWindow) void k_window_starts(uint32_t *counters, const uint32_t *__restrict__ tot,
                                                                Supers su, uint2 *__restrict__ starts) {
  constexpr int W = kSuperWindow / 64;
  __shared__ uint32_t s_p[kMostWindows][W], s_c[kMostWindows][W];
  if (counters[kCntPairs] == 0u) return;
  const int tid = threadIdx.x, windows = (su.n + kSuperWindow - 1) / kSuperWindow;
  for (int k = 0; k < windows; ++k) {
    const int s = k * kSuperWindow + tid;
    const uint32_t t = s < su.n ? tot[s] : 0u;
    const uint32_t p = wave_incl_scan(t), c = wave_incl_scan((t + kChunk - 1) / kChunk);
    if ((tid & 63) == 63) {
      s_p[k][tid >> 6] = p;
      s_c[k][tid >> 6] = c;
    }
  }
  __syncthreads();
  if (tid > windows) return;
  uint2 sum = make_uint2(0u, 0u);
  for (int k = 0; k < tid; ++k)
#pragma unroll
    for (int w = 0; w < W; ++w) {
      sum.x += s_p[k][w];
      sum.y += s_c[k][w];
    }
  if (tid < windows)
    starts[tid] = sum;
  else
    counters[kCntChunks] = sum.y;
}

// A 64 x 64 bit matrix, one row per lane (bit j of lane i), transposed: lane j gets column j
// (bit i from lane i). Six exchange steps between lanes k apart.
template <int K>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, (K << 10) | 0x1F);   // within 32 lanes
}

template <int K>
__device__ __forceinline__ uint32_t transpose_step(uint32_t x, uint32_t m, bool up) {
  const uint32_t y = lane_xor<K>(x);
  return up ? (x & ~m) | ((y & ~m) >> K) : (x & m) | ((y & m) << K);
}

__device__ __forceinline__ unsigned long long transpose64(unsigned long long v) {
  const int lane = threadIdx.x & 63;
  uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
  // 32 apart: a lane below 32 keeps its low word and takes its partner's as its high one
  const bool up = (lane & 32) != 0;
  const uint32_t got = __shfl_xor(up ? lo : hi, 32, 64);
  if (up)
    lo = got;
  else
    hi = got;
  uint32_t w[2] = {lo, hi};
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    uint32_t x = w[k];
    x = transpose_step<16>(x, 0x0000FFFFu, (lane & 16) != 0);
    x = transpose_step<8>(x, 0x00FF00FFu, (lane & 8) != 0);
    x = transpose_step<4>(x, 0x0F0F0F0Fu, (lane & 4) != 0);
    x = transpose_step<2>(x, 0x33333333u, (lane & 2) != 0);
    x = transpose_step<1>(x, 0x55555555u, (lane & 1) != 0);
    w[k] = x;
  }
  return ((unsigned long long)w[1] << 32) | w[0];
}

// ---------------------------------------------------------------------------------------
// Instances of each of the 64 tiles in each chunk of pairs: one wave per chunk, 64 pairs a
// round, the masks transposed so that lane t counts tile t.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_chunk_count(const uint32_t *__restrict__ counters,
                                                        const uint4 *__restrict__ chunks,
                                                        const unsigned long long *__restrict__ pair_mask,
                                                        uint32_t *__restrict__ cnt) {
  if (counters[kCntPairs] == 0u) return;
  const uint32_t nc = counters[kCntChunks];
  const uint32_t lane = threadIdx.x & 63;
  for (uint32_t c = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6); c < nc; c += gridDim.x * (kBlock / 64)) {
    const uint4 d = chunks[c];
    unsigned long long m[kChunk / 64];
#pragma unroll
    for (int r = 0; r < kChunk / 64; ++r) m[r] = r * 64 + lane < d.y ? pair_mask[d.x + r * 64 + lane] : 0ull;
    uint32_t acc = 0u;
#pragma unroll
    for (int r = 0; r < kChunk / 64; ++r) acc += (uint32_t)__popcll(transpose64(m[r]));
    cnt[(size_t)c * 64 + lane] = acc;
  }
}

// ---------------------------------------------------------------------------------------
// Per supertile (one workgroup): the chunk counts become their exclusive prefix over the
// supertile's chunks, the sums its tiles' list lengths. Lane t of every wave takes tile t, each
// wave a run of chunks.
// ---------------------------------------------------------------------------------------
constexpr int kPrefixThreads = 1024;

__global__ __launch_bounds__(kPrefixThreads) void k_chunk_prefix(const uint32_t *__restrict__ counters,
                                                                 const uint2 *__restrict__ supers, Supers su,
                                                                 uint32_t *__restrict__ cnt,
                                                                 uint32_t *__restrict__ tile_len) {
  constexpr int W = kPrefixThreads / 64, U = 8;
  __shared__ uint32_t s_sum[W][64];
  const int s = blockIdx.x;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint2 in = make_uint2(0u, 0u);
  if (counters[kCntPairs] != 0u) in = supers[s];
  const int n = (int)in.y, per = (n + W - 1) / W;
  const int r0 = min(n, w * per), r1 = min(n, r0 + per);
  uint32_t *row = cnt + (size_t)in.x * 64 + lane;
  uint32_t sum = 0u;
  for (int r = r0; r < r1; r += U) {
    uint32_t v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = r + u < r1 ? row[(size_t)(r + u) * 64] : 0u;
#pragma unroll
    for (int u = 0; u < U; ++u) sum += v[u];
  }
  s_sum[w][lane] = sum;
  __syncthreads();
  uint32_t run = 0u, total = 0u;
#pragma unroll
  for (int k = 0; k < W; ++k) {
    const uint32_t x = s_sum[k][lane];
    run += k < w ? x : 0u;
    total += x;
  }
  for (int r = r0; r < r1; r += U) {
    uint32_t v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = r + u < r1 ? row[(size_t)(r + u) * 64] : 0u;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (r + u < r1) row[(size_t)(r + u) * 64] = run;
      run += v[u];
    }
  }
  const int tx = (s % su.nx) * kSuper + (lane & 7), ty = (s / su.nx) * kSuper + (lane >> 3);
  if (w == 0 && tx < su.tiles_x && ty < su.tiles_y) tile_len[ty * su.tiles_x + tx] = total;
}

// The tiles' list ranges: the exclusive prefix of their lengths in tile order. Each workgroup takes
// kStartTiles tiles, two per thread, and sums the lengths of all tiles before them itself (at most
// 130 KB for 3840x2160, from L2), so that no workgroup waits for another; two adjacent tiles keep the
// stores whole (eight per thread in one workgroup took 31 us at 32,400 tiles and 8.8 at 8,160). Bound
// by latency: 4.8 and 4.5 us there, 2.5 at 64 tiles; 25, 8.9 and 7.2 as one workgroup that made the
// blend's order too.
constexpr int kStartTiles = 2 * kOrderThreads;

__global__ __launch_bounds__(kOrderThreads) void k_tile_starts(const uint32_t *__restrict__ tile_len, int n,
                                                               uint2 *__restrict__ ranges) {
  constexpr int W = kOrderThreads / 64, U = 8;
  __shared__ uint32_t s_before[W], s_own[W];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int base = (int)blockIdx.x * kStartTiles, t = base + 2 * tid;
  const uint32_t c0 = tile_len[min(t, n - 1)], c1 = tile_len[min(t + 1, n - 1)];   // those past the end go nowhere
  uint32_t before = 0u;
  for (int k = tid; k < base; k += kOrderThreads * U) {
    uint32_t v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = tile_len[min(k + u * kOrderThreads, base - 1)];   // in bounds: base < n
#pragma unroll
    for (int u = 0; u < U; ++u) before += k + u * kOrderThreads < base ? v[u] : 0u;
  }
  before = wave_incl_scan(before);
  const uint32_t incl = wave_incl_scan(c0 + c1);
  if (lane == 63) {
    s_before[w] = before;
    s_own[w] = incl;
  }
  lds_barrier();
  uint32_t at = incl - (c0 + c1);
#pragma unroll
  for (int k = 0; k < W; ++k) at += s_before[k] + (k < w ? s_own[k] : 0u);
  if (t < n) ranges[t] = make_uint2(at, at + c0);
  if (t + 1 < n) ranges[t + 1] = make_uint2(at + c0, at + c0 + c1);
}

// ---------------------------------------------------------------------------------------
// The list entries of one chunk (one workgroup): its masks transposed, each tile's pairs
// (their 8-bit index in the chunk) staged in LDS in order, then every tile's run written with
// consecutive stores by 16 lanes. 157.6M entries (631 MB, 92 us at the rate of a fill) in 208 us,
// 8.4M in 21 us, bound by VALU issue (placing the indices) and the two dependent LDS reads per
// entry. Chunks by xcd_block, so that the runs of a tile's consecutive chunks meet in one L2 (212
// against 220 us), the indices placed per 32-bit half (208). Waves storing each tile's entries
// by ballot, without LDS, took 230 us there and 28 for the 8.4M; runs begun at a 64-byte
// boundary 210 and 23.
// The first workgroups make the blend's tile order instead, which no other kernel before the blend needs: four
// waves for every kOrderTiles tiles, done within the expansion's time (the kernel unchanged at 157.6M, 8.4M and
// 0.7M entries) but where large frames show little (2k Gaussians at 3840x2160: 6 -> 39 us, 51 -> 44 with
// the ranges). One workgroup for all of a 16384x16384 frame's 1M tiles took 1,580 us of the kernel's, now 80 with the expansion.
// ---------------------------------------------------------------------------------------
constexpr int kOrderTiles = 32768;   // tiles per workgroup of the order (a 3840x2160 frame has 32,400)

__global__ __launch_bounds__(kChunk) void k_chunk_expand(const uint32_t *__restrict__ counters,
                                                         const uint4 *__restrict__ chunks,
                                                         const uint32_t *__restrict__ pair_id,
                                                         const unsigned long long *__restrict__ pair_mask,
                                                         const uint32_t *__restrict__ prefix,
                                                         const uint2 *__restrict__ ranges, Supers su,
                                                         uint32_t *__restrict__ values,
                                                         const uint32_t *__restrict__ tile_len, int n_tiles,
                                                         uint32_t *__restrict__ order, uint32_t n_order) {
  constexpr int W = kChunk / 64;
  __shared__ __align__(16) uint8_t s_stage[kChunk * 64];
  __shared__ uint32_t s_id[kChunk];
  __shared__ uint32_t s_cnt[W][64];
  __shared__ uint32_t s_lbase[64], s_len[64], s_gbase[64];
  if (blockIdx.x < n_order) {
    static_assert(sizeof(OrderShared<W>) <= sizeof(s_stage), "the order's LDS in place of the staged indices");
    const int first = (int)blockIdx.x, step = (int)n_order;
    tile_order<W>(CountCost{tile_len}, (n_tiles - first + step - 1) / step, order, TileSplit{0.0f, 0.0f, -1, -1},
                  *reinterpret_cast<OrderShared<W> *>(s_stage), first, step);
    return;
  }
  if (counters[kCntPairs] == 0u) return;
  const uint32_t nc = counters[kCntChunks];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  for (uint32_t c = xcd_block(blockIdx.x - n_order); c < nc; c += gridDim.x - n_order) {
    const uint4 d = chunks[c];
    const bool in = (uint32_t)tid < d.y;
    const unsigned long long m = in ? pair_mask[d.x + tid] : 0ull;
    s_id[tid] = in ? pair_id[d.x + tid] : 0u;
    if (w == 0) {
      const int s = (int)d.z;
      const int tx = (s % su.nx) * kSuper + (lane & 7), ty = (s / su.nx) * kSuper + (lane >> 3);
      const bool tile = tx < su.tiles_x && ty < su.tiles_y;
      s_gbase[lane] = tile ? ranges[ty * su.tiles_x + tx].x + prefix[(size_t)c * 64 + lane] : 0u;
    }
    unsigned long long col = transpose64(m);
    s_cnt[w][lane] = (uint32_t)__popcll(col);
    __syncthreads();
    uint32_t before = 0u, len = 0u;
#pragma unroll
    for (int k = 0; k < W; ++k) {
      const uint32_t x = s_cnt[k][lane];
      before += k < w ? x : 0u;
      len += x;
    }
    const uint32_t lbase = wave_incl_scan(len) - len;
    if (w == 0) {
      s_lbase[lane] = lbase;
      s_len[lane] = len;
    }
    uint8_t *out = s_stage + lbase + before;
    for (uint32_t x = (uint32_t)col; x; x &= x - 1u) *out++ = (uint8_t)(w * 64 + __builtin_ctz(x));
    for (uint32_t x = (uint32_t)(col >> 32); x; x &= x - 1u) *out++ = (uint8_t)(w * 64 + 32 + __builtin_ctz(x));
    __syncthreads();
    const int q = tid >> 4, l16 = tid & 15;
#pragma unroll
    for (int t0 = 0; t0 < 64; t0 += kChunk / 16) {
      const int t = t0 + q;
      const uint32_t nt = s_len[t], lb = s_lbase[t], gb = s_gbase[t];
      for (uint32_t e = l16; e < nt; e += 16) values[gb + e] = s_id[s_stage[lb + e]];
    }
    __syncthreads();   // the next chunk reuses the LDS
  }
}

// ---------------------------------------------------------------------------------------
// Totals of the preprocess's per-workgroup sums by themselves (after the buffers grew).
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_frame_totals(FrameTotals t) { frame_totals(t); }

// Tile id of every list entry (inspection): one workgroup per tile.
__global__ __launch_bounds__(kBlock) void k_tile_ids(const uint2 *__restrict__ ranges, uint32_t *__restrict__ tile_ids) {
  const uint2 r = ranges[blockIdx.x];
  for (uint32_t i = r.x + threadIdx.x; i < r.y; i += kBlock) tile_ids[i] = blockIdx.x;
}

// The binning record of each rendered candidate (inspection): mu', conic, support bound, rectangle.
__global__ __launch_bounds__(kBlock) void k_bin_records(int64_t n, const uint32_t *__restrict__ tiles,
                                                        const uint2 *__restrict__ rect, BinIn in,
                                                        float4 *__restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= n || tiles[i] == 0u) return;
  const uint2 r = rect[i];
  out[2 * i] = in.xyab[i];
  out[2 * i + 1] = make_float4(in.cop[i].x, in.qsup[i], __uint_as_float(r.x & ~(15u << kRectBefore)), __uint_as_float(r.y & kRectCorner));
}

static Supers supers_of(const DevCamera &cam) {
  Supers s;
  s.tiles_x = cam.tiles_x;
  s.tiles_y = cam.tiles_y;
  s.nx = (cam.tiles_x + kSuper - 1) / kSuper;
  s.n = s.nx * ((cam.tiles_y + kSuper - 1) / kSuper);
  return s;
}

static int super_windows(const Supers &su) { return (su.n + kSuperWindow - 1) / kSuperWindow; }

// Gaussians per column of the pair counts, of n candidates.
static uint32_t pair_column(const Supers &su, int64_t n) {
  if (su.n <= kSuperWindow) return kPairBlock;
  const int64_t blocks = (n + kPairBlock - 1) / kPairBlock;
  return (uint32_t)(kPairBlock * std::min<int64_t>(super_windows(su), (blocks + kColumnsMin - 1) / kColumnsMin));
}

static int64_t pair_columns(const Supers &su, int64_t n) {
  const uint32_t per = pair_column(su, n);
  return (n + per - 1) / per;
}

static int pair_stride(const Supers &su, int64_t n) { return (int)((pair_columns(su, n) + 7) & ~(int64_t)7); }

int super_count(const DevCamera &cam) { return supers_of(cam).n; }

size_t pair_hist_bytes(const DevCamera &cam, int64_t n) {
  const Supers su = supers_of(cam);
  return n > 0 ? 4 * (size_t)su.n * (size_t)pair_stride(su, n) : 0;
}

// the supertiles' totals, an even number of words, and the windows' starts
static size_t tot_words(const Supers &su) { return ((size_t)su.n + 1) & ~(size_t)1; }

size_t pair_tot_bytes(const DevCamera &cam) {
  const Supers su = supers_of(cam);
  return 4 * tot_words(su) + sizeof(uint2) * (size_t)super_windows(su);
}

int64_t chunk_capacity(const DevCamera &cam, int64_t pairs) { return pairs / kChunk + supers_of(cam).n; }

hipError_t launch_pair_offsets(const uint32_t *ids, const uint32_t *counters, const uint2 *srect, const BinIn &bin,
                               const DevCamera &cam, int64_t n, uint32_t *scan, uint32_t *tot, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const Supers su = supers_of(cam);
  const int stride = pair_stride(su, n);
  const uint32_t per = pair_column(su, n);
  hipLaunchKernelGGL(k_pair_hist, dim3(xcd_grid(pair_columns(su, n))), dim3(kPairBlock), 4 * (size_t)su.n, s, ids,
                     counters, srect, bin, su, scan, stride, per);
  return launch_row_scan(counters + kCntVisible, scan, scan, tot, su.n, stride, (int)per, s);
}

hipError_t launch_pair_place(const uint32_t *ids, uint32_t *counters, const uint2 *srect, const BinIn &bin,
                             const DevCamera &cam, int64_t n, const uint32_t *scan, uint32_t *tot,
                             uint32_t *pair_id, unsigned long long *pair_mask, uint4 *chunks, uint2 *supers,
                             hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const Supers su = supers_of(cam);
  const int windows = super_windows(su), stride = pair_stride(su, n);
  const unsigned columns = xcd_grid(pair_columns(su, n));
  uint2 *starts = reinterpret_cast<uint2 *>(tot + tot_words(su));
  if (windows > 1) {
    hipLaunchKernelGGL(k_window_starts, dim3(1), dim3(kSuperWindow), 0, s, counters, tot, su, starts);
    hipLaunchKernelGGL(k_pair_place<true>, dim3(columns, (unsigned)windows), dim3(kPairBlock), 0, s, ids, counters,
                       srect, bin, su, scan, tot, stride, pair_column(su, n), starts, pair_id, pair_mask, chunks, supers);
  } else {
    hipLaunchKernelGGL(k_pair_place<false>, dim3(columns), dim3(kPairBlock), 0, s, ids, counters, srect, bin, su, scan,
                       tot, stride, (uint32_t)kPairBlock, nullptr, pair_id, pair_mask, chunks, supers);
  }
  return hipGetLastError();
}

hipError_t launch_chunk_counts(const uint32_t *counters, const uint4 *chunks, const unsigned long long *pair_mask,
                               const uint2 *supers, const DevCamera &cam, int64_t max_chunks, uint32_t *cnt,
                               uint32_t *tile_len, hipStream_t s) {
  const Supers su = supers_of(cam);
  constexpr int per = kBlock / 64;
  // chunks beyond the grid are taken in turn: the grid is sized for the buffers' capacity, which
  // can far exceed the frame's chunks
  const int64_t grid = std::min<int64_t>((max_chunks + per - 1) / per, 4096);
  hipLaunchKernelGGL(k_chunk_count, dim3((unsigned)grid), dim3(kBlock), 0, s, counters,
                     chunks, pair_mask, cnt);
  hipLaunchKernelGGL(k_chunk_prefix, dim3((unsigned)su.n), dim3(kPrefixThreads), 0, s, counters, supers, su, cnt,
                     tile_len);
  return hipGetLastError();
}

hipError_t launch_tile_starts(const uint32_t *tile_len, int n_tiles, uint2 *ranges, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_tile_starts, dim3((unsigned)((n_tiles + kStartTiles - 1) / kStartTiles)), dim3(kOrderThreads),
                     0, s, tile_len, n_tiles, ranges);
  return hipGetLastError();
}

hipError_t launch_chunk_expand(const uint32_t *counters, const uint4 *chunks, const uint32_t *pair_id,
                               const unsigned long long *pair_mask, const uint32_t *prefix, const uint2 *ranges,
                               const DevCamera &cam, int64_t max_chunks, uint32_t *values, const uint32_t *tile_len,
                               uint32_t *order, hipStream_t s) {
  const int n_tiles = cam.tiles_x * cam.tiles_y;
  if (n_tiles <= 0) return hipSuccess;
  // without candidates the order alone
  const unsigned n_order = (unsigned)((n_tiles + kOrderTiles - 1) / kOrderTiles);
  const unsigned grid = n_order + xcd_grid(std::min<int64_t>(max_chunks, 8192));
  hipLaunchKernelGGL(k_chunk_expand, dim3(grid), dim3(kChunk), 0, s, counters, chunks, pair_id,
                     pair_mask, prefix, ranges, supers_of(cam), values, tile_len, n_tiles, order, n_order);
  return hipGetLastError();
}

hipError_t launch_frame_totals(const FrameTotals &t, hipStream_t s) {
  hipLaunchKernelGGL(k_frame_totals, dim3(1), dim3(kBlock), 0, s, t);
  return hipGetLastError();
}

hipError_t launch_bin_records(int64_t n, const uint32_t *tiles, const uint2 *rect, const BinIn &in, float4 *out,
                              hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_bin_records, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, n, tiles, rect, in,
                     out);
  return hipGetLastError();
}

hipError_t launch_tile_ids(const uint2 *ranges, int n_tiles, uint32_t *tile_ids, hipStream_t s) {
  if (n_tiles <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_tile_ids, dim3((unsigned)n_tiles), dim3(kBlock), 0, s, ranges, tile_ids);
  return hipGetLastError();
}

}  // namespace flod
