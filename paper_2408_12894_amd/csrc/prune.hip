// Overlap pruning (section Overlap Pruning): a Gaussian is removed when the mean distance to
// its three nearest other Gaussians, d_avg = (d_1 + d_2 + d_3) / 3, is below d_op.
//
// Only the decision d_avg < d_op is needed, and it depends on neighbours within R = 3 d_op
// alone: if the third-nearest lies at R or beyond, d_avg >= R / 3 = d_op and the Gaussian
// stays. So a uniform grid of cell edge c slightly above R (the search radius is widened by
// a relative 1e-9 so that the rounded comparison stays on the safe side) finds every
// neighbour that can matter in the 27 cells around a Gaussian's own.
//
//   1. cell of each mean (FP64 floor of x / c, clamped to 21 bits per axis: a monotone map,
//      so points closer than c along an axis stay in the same or adjacent cells), hashed by
//      blocks of cells to a table of T = 2^b >= n buckets (bucket_of); below
//      the bucket in the key, the Morton index of the point's subcell (3 bits for each of
//      up to three halvings of the cell);
//   2. stable radix sort of (key, index), then the means gathered into key order (16 B per
//      point, index in the fourth word), and per-bucket [start, end). The points of a subcell
//      of any level are then consecutive too: their runs go to an open-addressed table, for
//      the buckets and levels that are searched by subcell;
//   3. where points have few others in the 27 buckets around their own, a thread settles each
//      (k_prune_few). The others are searched by whole waves (k_prune_query), each group of points
//      sharing a subcell among the candidates of the finest level whose subcells hold about one point or more.
//      Every point within a subcell's edge lies in the searched subcells, so when the third
//      smallest distance found is below the edge the three are the true nearest; otherwise the
//      next coarser level is searched, down to the 27 cells. Squared distances are FP64, from
//      the FP32 means, summed x, y, z;
//   4. d_avg = ((d_1 + d_2) + d_3) / 3 in FP64 when d_3 < R (then these are the true three
//      nearest), +inf otherwise; keep = !(d_avg < d_op).
// Distances, their order of summation and the comparison are the same FP64 operations a
// brute-force evaluation performs, so the decisions match it bit for bit.
#include "flod_internal.h"

namespace flod {

constexpr int kCellBits = 21;
constexpr double kCellHalf = (double)(1 << (kCellBits - 1));

struct Grid {
  double inv_c;
  int shift;    // 64 - table bits
  int bits;     // table bits
  int levels;   // halvings of a cell the keys hold
};

// Halvings of a cell that fit the 32-bit keys and the run table's tags (one bit more).
constexpr int kPruneLevels = 3;

// A bucket of at least kSubcellMin[l - 1] points is searched by subcells of level l (the cell's
// edge / 2^l): from 12, 96 and 768 points its subcells of level 1, 2, 3 hold 1.5 or more on
// average and the sphere of their edge about six, so a first search mostly ends there.
// Buckets below are scanned whole. Their runs number at most 0.8 n: a bucket of m points has at
// most 8 runs of level 1 (m >= 12), 64 of level 2 (m >= 96) and 512 of level 3 (m >= 768).
__device__ __forceinline__ uint32_t subcell_min(int level) { return 12u << (3 * (level - 1)); }

__device__ __forceinline__ int32_t cell_of(float x, double inv_c) {
  double f = floor((double)x * inv_c);
  f = fmin(fmax(f, -kCellHalf), kCellHalf - 1.0);
  return (int32_t)f;
}

// A cell's bucket: 64 consecutive ones for each block of 4 x 4 x 4 cells, by the block's coordinates hashed
// (MurmurHash3's fmix64 finaliser), and in them the cell's place in the block, permuted by another part of the
// hash so that blocks on the same 64 meet evenly. The 27 cells around a point lie in at most
// eight blocks, so their ranges and points come from a few cache lines: each cell hashed by itself, all of
// flod_overlap_prune took 1,050 us for 1M points ten d_op apart and, one thread per point, 1,000, now 490.
__device__ __forceinline__ uint32_t bucket_of(int32_t ix, int32_t iy, int32_t iz, int shift) {
  const uint64_t m = (1ull << (kCellBits - 2)) - 1;
  const int32_t x = ix + (1 << (kCellBits - 1)), y = iy + (1 << (kCellBits - 1)), z = iz + (1 << (kCellBits - 1));
  uint64_t k = (((uint64_t)(x >> 2) & m) << (2 * kCellBits)) | (((uint64_t)(y >> 2) & m) << kCellBits) |
               ((uint64_t)(z >> 2) & m);
  k ^= k >> 33;
  k *= 0xff51afd7ed558ccdull;
  k ^= k >> 33;
  k *= 0xc4ceb9fe1a85ec53ull;
  k ^= k >> 33;
  const uint32_t in = (uint32_t)(x & 3) | ((uint32_t)(y & 3) << 2) | ((uint32_t)(z & 3) << 4);
  return ((uint32_t)(k >> (shift + 6)) << 6) | (in ^ ((uint32_t)k & 63u));
}

// Fine coordinate (eight per cell): its upper bits are cell_of's cell, since scaling by 8 is
// exact.
__device__ __forceinline__ int32_t fine_of(float x, double inv_c) {
  const double f = floor((double)x * inv_c * 8.0);
  return (int32_t)fmin(fmax(f, -8.0 * kCellHalf), 8.0 * kCellHalf - 1.0);
}

// Morton index of a subcell of level l from the low bits of fine coordinates >> (3 - l).
__device__ __forceinline__ uint32_t morton(uint32_t x, uint32_t y, uint32_t z, int l) {
  uint32_t m = 0u;
  for (int k = 0; k < l; ++k) m |= (((x >> k) & 1u) << (3 * k)) | (((y >> k) & 1u) << (3 * k + 1)) | (((z >> k) & 1u) << (3 * k + 2));
  return m;
}

// The keys; and what the steps behind them find cleared: the buckets' ranges, the run table's tags and the
// count of keys.
__global__ __launch_bounds__(kBlock) void k_prune_keys(const float *means, int64_t n, Grid g, uint32_t *keys,
                                                       uint32_t *vals, uint2 *ranges, uint32_t *tags,
                                                       uint32_t *counters) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= (int64_t)1 << g.bits) return;   // at least n
  ranges[i] = make_uint2(0u, 0u);
  if (g.levels > 0) tags[i] = 0u;
  if (i == 0) counters[kCntVisible] = (uint32_t)n;
  if (i >= n) return;
  const int32_t fx = fine_of(means[i * 3 + 0], g.inv_c);
  const int32_t fy = fine_of(means[i * 3 + 1], g.inv_c);
  const int32_t fz = fine_of(means[i * 3 + 2], g.inv_c);
  const int d = kPruneLevels - g.levels;
  keys[i] = (bucket_of(fx >> 3, fy >> 3, fz >> 3, g.shift) << (3 * g.levels)) |
            morton((uint32_t)(fx & 7) >> d, (uint32_t)(fy & 7) >> d, (uint32_t)(fz & 7) >> d, g.levels);
  vals[i] = (uint32_t)i;
}

// The size of the neighbour scan and the count of crowded points (k_prune_cost), in kPruneSums parts on
// cache lines of their own: added to one word each, the workgroups' atomics took 56 us for 500k points (31 for
// the size alone), in parts 20.
constexpr int kPruneSums = 16, kSumStride = 16;
static_assert(kPruneSums * kSumStride * sizeof(unsigned long long) <= kDepthRadix * sizeof(uint32_t), "in the sort's totals");

__global__ __launch_bounds__(kBlock) void k_prune_gather(const float *means, const uint32_t *sorted_vals, int64_t n,
                                                         float4 *pts, unsigned long long *sums) {
  const int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (p < kPruneSums * kSumStride) sums[p] = 0ull;
  if (p >= n) return;
  const uint32_t j = sorted_vals[p];
  pts[p] = make_float4(means[(int64_t)j * 3 + 0], means[(int64_t)j * 3 + 1], means[(int64_t)j * 3 + 2],
                       __uint_as_float(j));
}

// Run table: a run's tag is its key of bits + 3 l bits under a leading one, so the levels differ.
// Its 2^bits slots, of which at most 0.8 n <= 0.8 2^bits are taken, are probed in groups of four
// (one 16-byte load; slot by slot, a wave waited for the longest of its 64 probe sequences at
// each of 27 subcells).
__device__ __forceinline__ uint32_t run_group(uint32_t tag, int bits) { return (tag * 2654435769u) >> (34 - bits); }

__device__ __forceinline__ uint32_t run_tag(uint32_t key, int level, const Grid &g) {
  return (1u << (g.bits + 3 * level)) | (key >> (3 * (g.levels - level)));
}

// One thread per point in key order: the first and the last of a run find or take the run's
// slot and write its start and end.
__global__ __launch_bounds__(kBlock) void k_prune_runs(const uint32_t *__restrict__ keys,
                                                       const uint2 *__restrict__ ranges, int64_t n, Grid g,
                                                       uint32_t *__restrict__ tags, uint32_t *__restrict__ runs) {
  const int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (p >= n) return;
  const uint32_t key = keys[p];
  const uint32_t before = p > 0 ? keys[p - 1] : ~key, after = p + 1 < n ? keys[p + 1] : ~key;
  const uint2 r = ranges[key >> (3 * g.levels)];
  const uint32_t mask = (1u << (g.bits - 2)) - 1u;
  for (int l = 1; l <= g.levels && r.y - r.x >= subcell_min(l); ++l) {
    const int s = 3 * (g.levels - l);
    const bool first = (before >> s) != (key >> s) || p == 0, last = (after >> s) != (key >> s) || p + 1 == n;
    if (!first && !last) continue;
    const uint32_t tag = run_tag(key, l, g);
    uint32_t h = 4u * run_group(tag, g.bits);
    for (;;) {
      const uint32_t was = atomicCAS(&tags[h], 0u, tag);
      if (was == 0u || was == tag) break;
      h = (h & 3u) != 3u ? h + 1u : 4u * (((h >> 2) + 1u) & mask);
    }
    if (first) runs[2 * (size_t)h] = (uint32_t)p;
    if (last) runs[2 * (size_t)h + 1] = (uint32_t)(p + 1);
  }
}

// 64-bit value of a lane 1, 2, 4 or 8 further on in its row of 16 (cyclic).
template <int N>
__device__ __forceinline__ double row_ror64(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, 0x120 + N, 0xF, 0xF, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), 0x120 + N, 0xF, 0xF, true);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

__device__ __forceinline__ double row_min16(double v) {
  v = fmin(v, row_ror64<8>(v));
  v = fmin(v, row_ror64<4>(v));
  v = fmin(v, row_ror64<2>(v));
  return fmin(v, row_ror64<1>(v));
}

// d_avg from the three smallest squared distances, infinite unless they are within the radius.
__device__ __forceinline__ double mean_of_three(double d1, double d2, double d3, double radius) {
  const double d = sqrt(d3);
  return d < radius ? ((sqrt(d1) + sqrt(d2)) + d) / 3.0 : (double)INFINITY;
}

constexpr int kPruneHold = 192;   // candidates held in LDS at once

// One wave per `per` (at most 64) consecutive points in key order. The wave takes the points of one subcell after the other
// (of the level above the searched one, so that one set of candidates serves them all): lane i
// looks up the i-th of the 4 x 4 x 4 subcells around it (at level 0 the i-th of 27 cells), the
// candidates are gathered into LDS, and each row of 16 lanes goes through them for one point,
// every lane keeping the three smallest squared distances it meets; the row then draws the
// three smallest of all. Points not settled there are searched again one level coarser.
//
// Why so: one thread per point, walking its own 27 places, left a wave waiting at every place
// for its longest list and its slowest lookup (500k points at d_op 0.025, about 830 in the 27
// cells around each: 1.35 ms, 0.73 with subcells; this kernel 0.34 ms, VALU busy 62%, 228
// instructions per point).
__global__ __launch_bounds__(64) void k_prune_query(const float4 *__restrict__ pts, const uint2 *__restrict__ ranges,
                                                    const uint4 *__restrict__ tags, const uint2 *__restrict__ runs,
                                                    const uint32_t *__restrict__ around, int64_t n, int per, Grid g,
                                                    double radius, double d_op, const unsigned long long *cost,
                                                    uint8_t *keep, double *d_avg) {
  __shared__ double2 s_xy[kPruneHold];   // the candidates, converted once for all points
  __shared__ double s_z[kPruneHold];
  __shared__ uint32_t s_who[kPruneHold];
  __shared__ double s_best[64][3];
  __shared__ uint8_t s_lane[64];
  __shared__ uint32_t s_seen[128];
  if (*cost > kPruneMaxScan) return;   // refused: nothing is written
  const int lane = threadIdx.x, l16 = lane & 15, row = lane >> 4;
  const int64_t p = (int64_t)xcd_block(blockIdx.x) * per + lane;   // neighbours in key order share an XCD's L2
  const bool valid = lane < per && p < n && around[p] != 0u;   // 0: settled by k_prune_few
  const float4 a = valid ? pts[p] : make_float4(0.f, 0.f, 0.f, 0.f);
  const int fx = fine_of(a.x, g.inv_c), fy = fine_of(a.y, g.inv_c), fz = fine_of(a.z, g.inv_c);
  int level = 0;   // the point's level: the finest its own bucket's count allows
  bool pending = valid;
  if (pending) {
    const uint2 own = ranges[bucket_of(fx >> 3, fy >> 3, fz >> 3, g.shift)];
    while (level < g.levels && own.y - own.x >= subcell_min(level + 1)) ++level;
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) s_best[lane][k] = INFINITY;
  const unsigned long long below = lane ? (~0ull >> (64 - lane)) : 0ull;
  const uint32_t mask = (1u << (g.bits - 2)) - 1u;
  for (unsigned long long todo = __ballot(pending); todo; todo = __ballot(pending)) {
    // the group: the pending points of the first one's subcell and level
    const int src = __ffsll((long long)todo) - 1;
    const int l = __builtin_amdgcn_readlane(level, src);
    const int up = l > 0 ? kPruneLevels + 1 - l : kPruneLevels;   // fine coordinate >> up: the subcell
    const int gx = __builtin_amdgcn_readlane(fx, src) >> up, gy = __builtin_amdgcn_readlane(fy, src) >> up,
              gz = __builtin_amdgcn_readlane(fz, src) >> up;
    const bool in = pending && level == l && fx >> up == gx && fy >> up == gy && fz >> up == gz;
    const unsigned long long group = __ballot(in);
    const int count = __popcll(group);
    if (in) {
      s_lane[__popcll(group & below)] = (uint8_t)lane;
#pragma unroll
      for (int k = 0; k < 3; ++k) s_best[lane][k] = INFINITY;
    }
    // this lane's place and its run of points
    uint2 run = make_uint2(0u, 0u);
    if (l == 0) {
      if (lane < 27)
        run = ranges[bucket_of(gx + lane % 3 - 1, gy + (lane / 3) % 3 - 1, gz + lane / 9 - 1, g.shift)];
    } else {
      const int bx = 2 * gx - 1, by = 2 * gy - 1, bz = 2 * gz - 1;
      const int x = bx + (lane & 3), y = by + ((lane >> 2) & 3), z = bz + (lane >> 4);
      const uint32_t bucket = bucket_of(x >> l, y >> l, z >> l, g.shift);
      const uint2 r = ranges[bucket];
      // a bucket with fewer points has runs of a coarser level k, or is one run (k = 0): the
      // first of the places in it takes it
      int k = l;
      while (k > 0 && r.y - r.x < subcell_min(k)) --k;
      const int d = l - k, low = (1 << d) - 1;
      const bool first = ((x & low) == 0 || x == bx) && ((y & low) == 0 || y == by) && ((z & low) == 0 || z == bz);
      if (first && r.y != r.x) {
        if (k == 0) {
          run = r;
        } else {
          const uint32_t top = (1u << k) - 1u;
          const uint32_t tag = (1u << (g.bits + 3 * k)) | (bucket << (3 * k)) |
                               morton((uint32_t)(x >> d) & top, (uint32_t)(y >> d) & top, (uint32_t)(z >> d) & top, k);
          for (uint32_t h = run_group(tag, g.bits);; h = (h + 1u) & mask) {
            const uint4 w = tags[h];   // filled from the first slot on
            const uint32_t at = w.x == tag ? 0u : w.y == tag ? 1u : w.z == tag ? 2u : w.w == tag ? 3u : 4u;
            if (at < 4u) run = runs[4u * h + at];
            if (at < 4u || w.w == 0u) break;
          }
        }
      }
    }
    // two cells can share a bucket: of the lanes with the same run one keeps it (a lane is
    // settled when it wins its slot or meets its own run there)
    bool open = run.y > run.x;
    while (__any(open)) {
      const uint32_t slot = (run.x * 2654435769u) >> 25;
      if (open) s_seen[slot] = (uint32_t)lane;
      __syncthreads();
      const uint32_t who = open ? s_seen[slot] : (uint32_t)lane;
      const uint32_t its = __shfl(run.x, (int)who, 64);
      if (open && who != (uint32_t)lane && its == run.x) run.y = run.x;
      if (who == (uint32_t)lane || its == run.x) open = false;
      __syncthreads();
    }
    const uint32_t len = run.y - run.x;
    uint32_t end = len;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t t = __shfl_up(end, o, 64);
      if (lane >= o) end += t;
    }
    const uint32_t total = __shfl(end, 63, 64);
    const uint32_t shift = run.x - (end - len);   // candidate c of this lane's run is point c + shift
    for (uint32_t c0 = 0; c0 < total; c0 += kPruneHold) {
      const uint32_t held = min((uint32_t)kPruneHold, total - c0);
      for (uint32_t e = lane; e < ((held + 63u) & ~63u); e += 64) {
        // the lane whose run holds candidate c: the number of lanes with end <= c
        const uint32_t c = min(c0 + e, total - 1u);
        int o = 0;
#pragma unroll
        for (int step = 32; step > 0; step >>= 1)
          if (__shfl(end, o + step - 1, 64) <= c) o += step;
        const float4 b = pts[c + __shfl(shift, o, 64)];
        s_xy[e] = make_double2((double)b.x, (double)b.y);
        s_z[e] = (double)b.z;
        s_who[e] = __float_as_uint(b.w);
      }
      __syncthreads();
      for (int j0 = 0; j0 < count; j0 += 4) {
        const int j = j0 + row;
        const int who = s_lane[min(j, count - 1)];
        const double ax = __shfl(a.x, who, 64), ay = __shfl(a.y, who, 64), az = __shfl(a.z, who, 64);
        const uint32_t self = __float_as_uint(__shfl(a.w, who, 64));
        // the row's first lane starts from what earlier candidates gave
        double b0 = l16 == 0 ? s_best[who][0] : (double)INFINITY, b1 = l16 == 0 ? s_best[who][1] : (double)INFINITY,
               b2 = l16 == 0 ? s_best[who][2] : (double)INFINITY;
        for (uint32_t e = l16; e < held; e += 16) {
          const double2 b = s_xy[e];
          const double ex = b.x - ax, ey = b.y - ay, ez = s_z[e] - az;
          double d = fmin((ex * ex + ey * ey) + ez * ez, (double)INFINITY);   // NaN: infinite
          if (s_who[e] == self) d = INFINITY;
          const double t1 = fmax(b0, d), t2 = fmax(b1, t1);
          b0 = fmin(b0, d);
          b1 = fmin(b1, t1);
          b2 = fmin(b2, t2);
        }
        double best[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          best[k] = row_min16(b0);
          // the first lane of the row that holds it gives it up
          const uint32_t hold = (uint32_t)(__ballot(b0 == best[k]) >> (16 * row)) & 0xFFFFu;
          if (l16 == __ffs((int)hold) - 1) {
            b0 = b1;
            b1 = b2;
            b2 = INFINITY;
          }
        }
        if (l16 == 0 && j < count) {
#pragma unroll
          for (int k = 0; k < 3; ++k) s_best[who][k] = best[k];
        }
      }
      __syncthreads();
    }
    // the edge of a subcell is above radius / 2^l (see make_grid), so nothing nearer is outside
    const double edge = radius / (double)(1 << l);
    if (in) {
      pending = l > 0 && !(s_best[lane][2] < edge * edge);
      level = l - 1;
    }
  }
  if (!valid) return;
  const double avg = mean_of_three(s_best[lane][0], s_best[lane][1], s_best[lane][2], radius);
  const uint32_t j = __float_as_uint(a.w);
  keep[j] = (avg < d_op) ? 0 : 1;
  if (d_avg) d_avg[j] = avg;
}

constexpr uint32_t kPruneFew = 320;

// Size of the neighbour scan over whole cells: per point its 27 buckets' occupancy (to around),
// and in parts their sum and the count of those above kPruneFew.
__global__ __launch_bounds__(kBlock) void k_prune_cost(const float4 *__restrict__ pts, const uint2 *__restrict__ ranges,
                                                       int64_t n, Grid g, uint32_t *__restrict__ around,
                                                       unsigned long long *sums) {
  __shared__ unsigned long long s_sum[kBlock / 64];
  __shared__ uint32_t s_crowd[kBlock / 64];
  const int64_t p = (int64_t)xcd_block(blockIdx.x) * kBlock + threadIdx.x;
  unsigned long long c = 0;
  if (p < n) {
    const float4 a = pts[p];
    const int32_t cx = cell_of(a.x, g.inv_c), cy = cell_of(a.y, g.inv_c), cz = cell_of(a.z, g.inv_c);
    for (int dz = -1; dz <= 1; ++dz)
      for (int dy = -1; dy <= 1; ++dy)
        for (int dx = -1; dx <= 1; ++dx) {
          const uint2 r = ranges[bucket_of(cx + dx, cy + dy, cz + dz, g.shift)];
          c += r.y - r.x;
        }
    around[p] = (uint32_t)(c < 0xFFFFFFFFull ? c : 0xFFFFFFFFull);
  }
  const uint32_t crowd = (uint32_t)__popcll(__ballot(c > kPruneFew));
  for (int o = 32; o > 0; o >>= 1) c += __shfl_down(c, o, 64);
  if ((threadIdx.x & 63) == 0) {
    s_sum[threadIdx.x >> 6] = c;
    s_crowd[threadIdx.x >> 6] = crowd;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long t = 0, m = 0;
    for (int w = 0; w < kBlock / 64; ++w) {
      t += s_sum[w];
      m += s_crowd[w];
    }
    unsigned long long *part = sums + (blockIdx.x % kPruneSums) * kSumStride;
    atomicAdd(&part[0], t);
    if (m) atomicAdd(&part[1], m);
  }
}

// One thread per point where few points lie around: of kPruneFewFrom points or more (fewer leave most of the
// device idle in long chains) of which at most one in 256 has more than kPruneFew in its 27 buckets, those
// with that many or fewer are settled here, else those alone that have fewer than three others there. around is set to 0
// for k_prune_query, whose waves take the points of one cell after the other, which costs where
// they are few to a cell. A choice for the call as a whole: waves that find
// some of their points settled take hardly less time. kTogether cells at a time: their ranges and
// then their first points are loaded together.
// All of flod_overlap_prune in us, points at random f d_op apart, one thread per point throughout | by
// waves alone (each without the block hash) | now:
//   300k, f = 10, 3, 2, 1     245 240 264 490 | 361 315 284 276 | 194 207 243 269
//   1M                        960 743 551 1044 | 1044 819 617 687 | 486 379 535 557
constexpr int64_t kPruneFewFrom = 32768;

__global__ __launch_bounds__(kBlock) void k_prune_few(const float4 *__restrict__ pts, const uint2 *__restrict__ ranges,
                                                      uint32_t *__restrict__ around, int64_t n, Grid g, double radius,
                                                      double d_op, const unsigned long long *sums,
                                                      unsigned long long *cost, uint8_t *keep, double *d_avg) {
  constexpr int kTogether = 4;
  __shared__ unsigned long long s_sum[2];
  if (threadIdx.x < 64) {
    const bool in = threadIdx.x < kPruneSums;
    unsigned long long t = in ? sums[threadIdx.x * kSumStride] : 0ull, m = in ? sums[threadIdx.x * kSumStride + 1] : 0ull;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      t += __shfl_xor(t, o, 64);
      m += __shfl_xor(m, o, 64);
    }
    if (threadIdx.x == 0) {
      s_sum[0] = t;
      s_sum[1] = m;
      if (blockIdx.x == 0) *cost = t;   // for k_prune_query and the host
    }
  }
  __syncthreads();
  if (s_sum[0] > kPruneMaxScan) return;   // refused: nothing is written
  const int64_t p = (int64_t)xcd_block(blockIdx.x) * kBlock + threadIdx.x;
  if (p >= n) return;
  const uint32_t c = around[p];
  if (c > (n >= kPruneFewFrom && s_sum[1] <= (unsigned long long)n / 256u ? kPruneFew : 3u)) return;
  const float4 a = pts[p];
  double avg = INFINITY;
  if (c > 3u) {
    const double ax = a.x, ay = a.y, az = a.z;
    const int32_t cx = cell_of(a.x, g.inv_c), cy = cell_of(a.y, g.inv_c), cz = cell_of(a.z, g.inv_c);
    // the three smallest squared distances below the radius' and their points: a point met again, in a
    // bucket that two of the cells share, is one of them or no nearer than they are
    const double reach = radius * radius * (1.0 + 1e-12);
    double b0 = reach, b1 = reach, b2 = reach;
    uint32_t q0 = (uint32_t)p, q1 = q0, q2 = q0;
    const auto meet = [&](uint32_t q, const float4 &b) {
      const double ex = (double)b.x - ax, ey = (double)b.y - ay, ez = (double)b.z - az;
      const double d = (ex * ex + ey * ey) + ez * ez;
      if (!(d < b2) || q == (uint32_t)p || q == q0 || q == q1 || q == q2) return;
      const bool first = d < b0, second = d < b1;
      b2 = second ? b1 : d;
      q2 = second ? q1 : q;
      b1 = first ? b0 : second ? d : b1;
      q1 = first ? q0 : second ? q : q1;
      b0 = first ? d : b0;
      q0 = first ? q : q0;
    };
    const auto bucket = [&](int k) { return bucket_of(cx + k % 3 - 1, cy + (k / 3) % 3 - 1, cz + k / 9 - 1, g.shift); };
    for (int k0 = 0; k0 < 27; k0 += kTogether) {
      uint2 r[kTogether];
      float4 first[kTogether];
#pragma unroll
      for (int i = 0; i < kTogether; ++i) r[i] = k0 + i < 27 ? ranges[bucket(k0 + i)] : make_uint2(0u, 0u);
#pragma unroll
      for (int i = 0; i < kTogether; ++i) first[i] = pts[r[i].y > r[i].x ? r[i].x : (uint32_t)p];
#pragma unroll
      for (int i = 0; i < kTogether; ++i) {
        if (r[i].y > r[i].x) meet(r[i].x, first[i]);
        for (uint32_t q = r[i].x + 1; q < r[i].y; q += kTogether) {
          float4 b[kTogether];
#pragma unroll
          for (int u = 0; u < kTogether; ++u) b[u] = pts[min(q + u, r[i].y - 1u)];
#pragma unroll
          for (int u = 0; u < kTogether; ++u)
            if (q + u < r[i].y) meet(q + u, b[u]);
        }
      }
    }
    avg = mean_of_three(b0, b1, b2, radius);
  }
  around[p] = 0u;
  const uint32_t j = __float_as_uint(a.w);
  keep[j] = (avg < d_op) ? 0 : 1;
  if (d_avg) d_avg[j] = avg;
}

__global__ __launch_bounds__(kBlock) void k_prune_none(int64_t n, uint8_t *keep, double *d_avg) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  keep[i] = 1;
  if (d_avg) d_avg[i] = INFINITY;
}

static unsigned grid_of(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

int prune_table_bits(int64_t n) {
  int b = 8;
  while (b < 31 && ((int64_t)1 << b) < n) ++b;
  return b;
}

// Halvings of a cell in the keys: a run's tag of bits + 3 levels + 1 bits fits 32. None for up to 256 points,
// whose keys then take one pass of the sort instead of three (20 points: 78 instead of 94 us in all).
int prune_levels(int64_t n) {
  if (n <= kRadix) return 0;
  const int l = (31 - prune_table_bits(n)) / 3;
  return l < kPruneLevels ? l : kPruneLevels;
}

static Grid make_grid(double radius, int64_t n) {
  Grid g;
  g.inv_c = 1.0 / (radius * 1.001);
  g.bits = prune_table_bits(n);
  g.shift = 64 - g.bits;
  g.levels = prune_levels(n);
  return g;
}

double prune_radius(float d_op) { return 3.0 * (double)d_op * (1.0 + 1e-9); }

hipError_t launch_prune_keys(const float *means, int64_t n, float d_op, uint32_t *keys, uint32_t *vals, uint2 *ranges,
                             uint32_t *tags, uint32_t *counters, hipStream_t s) {
  if (n <= 0 || !(d_op > 0.0f)) return hipSuccess;
  const Grid g = make_grid(prune_radius(d_op), n);
  hipLaunchKernelGGL(k_prune_keys, dim3(grid_of((int64_t)1 << g.bits)), dim3(kBlock), 0, s, means, n, g, keys, vals,
                     ranges, tags, counters);
  return hipGetLastError();
}

hipError_t launch_prune_gather(const float *means, const uint32_t *sorted_vals, int64_t n, float4 *pts,
                               unsigned long long *sums, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_prune_gather, dim3(grid_of(n)), dim3(kBlock), 0, s, means, sorted_vals, n, pts, sums);
  return hipGetLastError();
}

hipError_t launch_prune_cost(const float4 *pts, const uint2 *ranges, int64_t n, float d_op, uint32_t *around,
                             unsigned long long *sums, hipStream_t s) {
  if (n <= 0 || !(d_op > 0.0f)) return hipSuccess;
  hipLaunchKernelGGL(k_prune_cost, dim3(xcd_grid((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, pts, ranges, n,
                     make_grid(prune_radius(d_op), n), around, sums);
  return hipGetLastError();
}

hipError_t launch_prune_runs(const uint32_t *keys, const uint2 *ranges, int64_t n, float d_op, uint32_t *tags,
                             uint2 *runs, hipStream_t s) {
  if (n <= 0 || !(d_op > 0.0f)) return hipSuccess;
  const Grid g = make_grid(prune_radius(d_op), n);
  if (g.levels == 0) return hipSuccess;
  hipLaunchKernelGGL(k_prune_runs, dim3(grid_of(n)), dim3(kBlock), 0, s, keys, ranges, n, g, tags,
                     reinterpret_cast<uint32_t *>(runs));
  return hipGetLastError();
}

hipError_t launch_prune_query(const float4 *pts, const uint2 *ranges, const uint32_t *tags, const uint2 *runs,
                              uint32_t *around, int64_t n, float d_op, const unsigned long long *sums,
                              unsigned long long *cost, uint8_t *keep, double *d_avg, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (!(d_op > 0.0f)) {
    hipLaunchKernelGGL(k_prune_none, dim3(grid_of(n)), dim3(kBlock), 0, s, n, keep, d_avg);
    return hipGetLastError();
  }
  const double radius = prune_radius(d_op);
  hipLaunchKernelGGL(k_prune_few, dim3(xcd_grid((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, pts, ranges, around, n,
                     make_grid(radius, n), radius, (double)d_op, sums, cost, keep, d_avg);
  // points per wave: a wave takes its groups one after the other, each a chain of lookups, so
  // few points are spread over as many waves as the device holds (about 8,192): 69.6k points
  // at d_op 0.0125, mostly alone in their cell, take 50 us at 8 per wave, about 120 at 64
  int per = 64;
  while (per > 8 && n < (int64_t)per * 8192) per /= 2;
  hipLaunchKernelGGL(k_prune_query, dim3(xcd_grid((n + per - 1) / per)), dim3(64), 0, s, pts, ranges,
                     reinterpret_cast<const uint4 *>(tags), runs, around, n, per,
                     make_grid(radius, n), radius, (double)d_op, cost, keep, d_avg);
  return hipGetLastError();
}

}  // namespace flod
