// Sorting and scans: the stable radix sort (of the visible Gaussians by depth, and of the overlap
// pruning's points by bucket), row scans of counts and bucket ranges.
//
// A frame of up to kSmallSort candidates is depth-sorted by one workgroup. Else the depth sort's
// first pass reads every candidate's depth key in index order and drops the
// candidates not rendered (key kDepthNone), so it also compacts the visible set.
//
// The radix pass is a reduce-then-scan design (no inter-workgroup spinning, which would
// need cross-XCD coherent flags): per-workgroup digit histograms, a per-digit scan over
// workgroups, then a scatter in which each workgroup ranks its 2048 (3072, 4096) keys stably in LDS
// (wave64 ballots over the digit bits), reorders them by digit in LDS and writes each
// digit run contiguously.
#include <algorithm>
#include <type_traits>

#include "project.h"

namespace flod {

// Exclusive scan over a kBlock-thread workgroup; *total receives the sum.
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t *total) {
  __shared__ uint32_t s_w[kBlock / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t inc = wave_incl_scan(v);
  if (lane == 63) s_w[w] = inc;
  __syncthreads();
  uint32_t base = 0, tot = 0;
#pragma unroll
  for (int k = 0; k < kBlock / 64; ++k) {
    uint32_t t = s_w[k];
    base += (k < w) ? t : 0u;
    tot += t;
  }
  __syncthreads();
  *total = tot;
  return base + inc - v;
}

// ---------------------------------------------------------------------------------------
// Scans of per-workgroup counts, one workgroup each: 64-bit exclusive prefixes and the total; with
// host_out (coherent host memory) the total also goes there, tagged as the frame's counts are
// (see FrameTotals), and behind it, when given, the low and high halves of *extra.
// ---------------------------------------------------------------------------------------
constexpr int kScanThreads = 1024;

__global__ __launch_bounds__(kScanThreads) void k_scan_blocks(ScanJobs jobs, uint32_t host_seq,
                                                              const unsigned long long *extra) {
  __shared__ unsigned long long s_w[kScanThreads / 64];
  const ScanJob job = jobs.job[blockIdx.x];
  const uint32_t *in = job.in;
  unsigned long long *prefix = job.prefix, *host_out = job.host_out;
  const int nb = job.blocks;
  // thread t owns the contiguous counts [t per, (t + 1) per): its sum, a workgroup scan of the
  // sums, then its exclusive prefixes (a second read of its counts, from cache)
  const int per = (nb + kScanThreads - 1) / kScanThreads;
  const int lo = min(nb, (int)threadIdx.x * per), hi = min(nb, lo + per);
  // up to kScanHeld counts per thread are loaded together and kept for the prefixes (one memory
  // round trip instead of one per count); more (above kScanHeld x 1024 workgroups) are re-read
  constexpr int kScanHeld = 8;
  uint32_t held[kScanHeld];
#pragma unroll
  for (int i = 0; i < kScanHeld; ++i) held[i] = lo + i < hi ? in[lo + i] : 0u;
  unsigned long long mine = 0;
#pragma unroll
  for (int i = 0; i < kScanHeld; ++i) mine += held[i];
  for (int k = lo + kScanHeld; k < hi; ++k) mine += in[k];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  unsigned long long inc = mine;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const unsigned long long t = __shfl_up(inc, o, 64);
    if (lane >= o) inc += t;
  }
  if (lane == 63) s_w[w] = inc;
  __syncthreads();
  unsigned long long run = inc - mine, total = 0;
#pragma unroll
  for (int k = 0; k < kScanThreads / 64; ++k) {
    const unsigned long long t = s_w[k];
    run += (k < w) ? t : 0ull;
    total += t;
  }
#pragma unroll
  for (int i = 0; i < kScanHeld; ++i) {
    if (lo + i < hi) prefix[lo + i] = run;
    run += held[i];
  }
  for (int k = lo + kScanHeld; k < hi; ++k) {
    prefix[k] = run;
    run += in[k];
  }
  if (threadIdx.x == 0) {
    *job.total = (uint32_t)total;
    if (host_out) {
      const unsigned long long tag = (unsigned long long)host_seq << 32, x = extra ? *extra : 0ull;
      const unsigned long long w[3] = {tag | (uint32_t)total, tag | (uint32_t)x, tag | (x >> 32)};
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if (k == 0 || extra) __hip_atomic_store(&host_out[k], w[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
  }
}

hipError_t launch_scan_blocks(const ScanJobs &jobs, int n_jobs, uint32_t host_seq, hipStream_t s,
                              const unsigned long long *extra) {
  hipLaunchKernelGGL(k_scan_blocks, dim3((unsigned)n_jobs), dim3(kScanThreads), 0, s, jobs, host_seq, extra);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Radix pass: histogram, per-digit scan, stable scatter.
// hist[d * stride + b] = count of digit d in block b; scan = exclusive prefix over b. The row
// stride is the block count rounded up to a multiple of 8 (32-byte aligned rows). Workgroups
// take their block by xcd_block.
// ---------------------------------------------------------------------------------------
// All of a workgroup's keys are loaded before the first LDS update, so its loads are in
// flight together. The count n is read first: grids are sized for the buffers' capacity,
// which can far exceed n, and workgroups past n leave without reading their keys.
//
// FIRST (the depth sort's first pass): the keys are all n_all candidates' depth keys, read
// directly, and keys equal to kDepthNone (candidates not rendered) are not counted. Each
// workgroup also adds up the preprocess's counts of its ITEMS workgroups (sums to part), so that
// the one workgroup that takes the totals reads ITEMS times fewer (alone over all 17,149 of a
// 4.39M-Gaussian stack it took 22 us).
template <int RB, int ITEMS, bool FIRST>
__global__ __launch_bounds__(kBlock) void k_rs_hist(const uint32_t *keys, const uint32_t *n_ptr, uint32_t n_all,
                                                    int shift, uint32_t dmask, uint32_t *hist, int stride,
                                                    const uint4 *__restrict__ sums, uint4 *__restrict__ part) {
  constexpr uint32_t TILE = kBlock * ITEMS;
  static_assert(ITEMS <= 64, "one wave adds a workgroup's counts");
  constexpr int DIGITS = 1 << RB;
  __shared__ uint32_t h[DIGITS];
  const uint32_t n = FIRST ? n_all : *n_ptr;
  const uint32_t nb = (n + TILE - 1) / TILE;
  const uint32_t b = xcd_block(blockIdx.x);
  if (b >= nb) return;
  const uint32_t base = b * TILE;
  uint32_t kr[ITEMS];
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const uint32_t idx = base + r * kBlock + threadIdx.x;
    kr[r] = idx < n ? keys[idx] : 0u;
  }
#pragma unroll
  for (int k = 0; k < DIGITS; k += kBlock) h[k + threadIdx.x] = 0;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ITEMS; ++r)
    if (base + r * kBlock + threadIdx.x < n && (!FIRST || kr[r] != kDepthNone))
      atomicAdd(&h[((FIRST ? kr[r] - kDepthBase : kr[r]) >> shift) & dmask], 1u);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < DIGITS; k += kBlock) hist[(size_t)(k + threadIdx.x) * stride + b] = h[k + threadIdx.x];
  if (FIRST && threadIdx.x < 64) {
    const uint32_t i = b * ITEMS + threadIdx.x;
    uint4 x = make_uint4(0u, 0u, 0u, 0u);
    if (threadIdx.x < ITEMS && i < (n + kBlock - 1) / kBlock) x = sums[i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      x.x += __shfl_xor(x.x, o, 64);
      x.y += __shfl_xor(x.y, o, 64);
      x.z += __shfl_xor(x.z, o, 64);
      x.w += __shfl_xor(x.w, o, 64);
    }
    if (threadIdx.x == 0) part[b] = x;
  }
}

// One workgroup per row (digit). Rounds of 2048 counts: each thread takes 8 consecutive ones (two
// 16-byte loads), the next round's loads are issued before this round's scan. TOTALS (the depth
// sort's first pass): one workgroup more, which takes the frame's totals beside the rows.
template <bool TOTALS>
__global__ __launch_bounds__(kBlock) void k_rs_scan(const uint32_t *n_ptr, uint32_t n_all, const uint32_t *hist,
                                                    uint32_t *scan, uint32_t *tot, int stride, int tile,
                                                    FrameTotals totals) {
  if (TOTALS && blockIdx.x == gridDim.x - 1) {
    frame_totals(totals);
    return;
  }
  constexpr uint32_t kPer = 8, kRound = kBlock * kPer;
  const uint32_t n = n_ptr ? *n_ptr : n_all;   // null: the first pass over all candidates
  const uint32_t nb = (n + tile - 1) / tile;
  const int d = blockIdx.x;
  const uint32_t *row = hist + (size_t)d * stride;
  uint32_t *out = scan + (size_t)d * stride;
  // k < nb implies k + 3 < stride: a 16-byte group that starts below nb lies inside the row
  auto load = [&](uint32_t k, uint4 &lo, uint4 &hi) {
    const uint4 z = make_uint4(0u, 0u, 0u, 0u);
    lo = k < nb ? *reinterpret_cast<const uint4 *>(row + k) : z;
    hi = k + 4 < nb ? *reinterpret_cast<const uint4 *>(row + k + 4) : z;
  };
  uint32_t run = 0;
  uint32_t k = threadIdx.x * kPer;
  uint4 lo, hi;
  load(k, lo, hi);
  for (uint32_t base = 0; base < nb; base += kRound, k += kRound) {
    uint32_t v[kPer] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    load(k + kRound, lo, hi);
    uint32_t sum = 0;
#pragma unroll
    for (uint32_t i = 0; i < kPer; ++i) {
      if (k + i >= nb) v[i] = 0u;
      sum += v[i];
    }
    uint32_t t;
    uint32_t e = run + block_excl_scan(sum, &t);
    uint32_t o[kPer];
#pragma unroll
    for (uint32_t i = 0; i < kPer; ++i) {
      o[i] = e;
      e += v[i];
    }
    if (k < nb) *reinterpret_cast<uint4 *>(out + k) = make_uint4(o[0], o[1], o[2], o[3]);
    if (k + 4 < nb) *reinterpret_cast<uint4 *>(out + k + 4) = make_uint4(o[4], o[5], o[6], o[7]);
    run += t;
  }
  if (threadIdx.x == 0) tot[d] = run;
}

// Stable scatter of one workgroup's TILE keys. Wave w owns the contiguous keys
// [w * 64 ITEMS, (w + 1) * 64 ITEMS) of the tile, read round by round (64 consecutive keys per
// round), so (wave, round, lane) order is the input order. Each key's rank among equal digits
// of its wave comes from ballots over the digit bits plus a wave-private LDS count carried
// across rounds (a wave's LDS accesses complete in program order, so no barrier is needed
// between rounds); one barrier then turns the per-wave counts into offsets, keys are placed
// in LDS in digit order, and each digit's run is written out contiguously.
//
// With RECTS (the last pass of the depth sort) the scatter also writes, at each output
// position, the tile rectangle of the Gaussian its value names (rect_out[pos] = rect_of[val]).
//
// With FIRST (the depth sort's first pass) the keys are all n_all candidates' depth keys, each
// key's value is its index, keys equal to kDepthNone are dropped (the output is the rendered
// candidates, compacted and ordered by the first digit), and workgroup 0 writes the count kept
// to *n_out for the later passes.
template <int RB, int ITEMS, bool RECTS, bool FIRST>
__global__ __launch_bounds__(kBlock) void k_rs_scatter(const uint32_t *__restrict__ keys_in,
                                                       const uint32_t *__restrict__ vals_in,
                                                       uint32_t *__restrict__ keys_out,
                                                       uint32_t *__restrict__ vals_out, const uint32_t *n_ptr,
                                                       uint32_t n_all, uint32_t *n_out, int shift, uint32_t dmask,
                                                       const uint32_t *hist, const uint32_t *scan,
                                                       const uint32_t *tot, int stride,
                                                       const uint2 *__restrict__ rect_of,
                                                       uint2 *__restrict__ rect_out) {
  constexpr uint32_t TILE = kBlock * ITEMS;
  constexpr int WAVES = kBlock / 64;
  constexpr uint32_t WTILE = 64 * ITEMS;
  constexpr int DIGITS = 1 << RB, DP = DIGITS / kBlock;   // thread t has digits DP t .. DP t + DP - 1
  __shared__ uint32_t s_keys[TILE];
  __shared__ uint32_t s_vals[TILE];
  __shared__ uint32_t s_goff[DIGITS];
  __shared__ uint32_t s_wcnt[WAVES][DIGITS];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  // the count first (grids are sized for the capacity, which can far exceed it); then the
  // tile's keys and values, loaded together with the digit offsets below, so that their
  // latencies overlap (ahead of the count, a wait for it would wait for the scattered offset rows too)
  const uint32_t n = FIRST ? n_all : *n_ptr;
  const uint32_t nb = (n + TILE - 1) / TILE;
  const uint32_t b = xcd_block(blockIdx.x);
  if (b >= nb) return;
  const uint32_t base = b * TILE;
  const uint32_t count = min(TILE, n - base);
  uint32_t kr[ITEMS], vr[ITEMS], rr[ITEMS];
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const uint32_t li = (uint32_t)w * WTILE + (uint32_t)r * 64u + (uint32_t)lane;
    kr[r] = li < count ? keys_in[base + li] : (FIRST ? kDepthNone : 0u);
    if (FIRST && kr[r] != kDepthNone) kr[r] -= kDepthBase;
    vr[r] = FIRST ? base + li : (li < count ? vals_in[base + li] : 0u);
  }
  // digit bases over the whole array and this workgroup's local digit bases (the
  // loads issued together, ahead of the scans' barriers)
  uint32_t tot_d[DP], cnt[DP], sc[DP], sum_t = 0u, sum_c = 0u;
#pragma unroll
  for (int k = 0; k < DP; ++k) {
    const int d = DP * tid + k;
    tot_d[k] = tot[d];
    cnt[k] = hist[(size_t)d * stride + b];
    sc[k] = scan[(size_t)d * stride + b];
  }
#pragma unroll
  for (int k = 0; k < DP; ++k) {
    sum_t += tot_d[k];
    sum_c += cnt[k];
  }
  uint32_t t_all;
  uint32_t dbase = block_excl_scan(sum_t, &t_all);
  uint32_t t_loc;   // the keys this workgroup writes (FIRST: the rendered ones)
  const uint32_t lbase = block_excl_scan(sum_c, &t_loc);
  if (FIRST && b == 0 && tid == 0) *n_out = t_all;
  uint32_t lb = lbase;
#pragma unroll
  for (int k = 0; k < DP; ++k) {
    s_goff[DP * tid + k] = dbase + sc[k] - lb;
    dbase += tot_d[k];
    lb += cnt[k];
  }
#pragma unroll
  for (int k = 0; k < WAVES; ++k)
#pragma unroll
    for (int d = 0; d < DIGITS; d += kBlock) s_wcnt[k][d + tid] = 0;
  __syncthreads();
  const unsigned long long lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const uint32_t li = (uint32_t)w * WTILE + (uint32_t)r * 64u + (uint32_t)lane;
    const bool valid = li < count && (!FIRST || kr[r] != kDepthNone);
    const uint32_t key = kr[r];
    const uint32_t d = (key >> shift) & dmask;   // bits above the pass's digit are zero
    unsigned long long peers = __ballot(valid);
#pragma unroll
    for (int bit = 0; bit < RB; ++bit) {
      const bool set = (d >> bit) & 1u;
      const unsigned long long bb = __ballot(set);
      peers &= set ? bb : ~bb;
    }
    const uint32_t in_round = (uint32_t)__popcll(peers & lt);
    const uint32_t prev = s_wcnt[w][d];
    rr[r] = prev + in_round;
    if (valid && in_round == 0) s_wcnt[w][d] = prev + (uint32_t)__popcll(peers);
  }
  __syncthreads();
  {
    uint32_t acc = lbase;
#pragma unroll
    for (int j = 0; j < DP; ++j)
#pragma unroll
      for (int k = 0; k < WAVES; ++k) {
        const uint32_t c = s_wcnt[k][DP * tid + j];
        s_wcnt[k][DP * tid + j] = acc;
        acc += c;
      }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const uint32_t li = (uint32_t)w * WTILE + (uint32_t)r * 64u + (uint32_t)lane;
    if (li < count && (!FIRST || kr[r] != kDepthNone)) {
      const uint32_t pos = s_wcnt[w][(kr[r] >> shift) & dmask] + rr[r];
      s_keys[pos] = kr[r];
      s_vals[pos] = vr[r];
    }
  }
  __syncthreads();
  const uint32_t kept = FIRST ? t_loc : count;
  for (uint32_t li = tid; li < kept; li += kBlock) {
    const uint32_t key = s_keys[li];
    const uint32_t val = s_vals[li];
    const uint32_t pos = s_goff[(key >> shift) & dmask] + li;
    keys_out[pos] = key;
    vals_out[pos] = val;
    if (RECTS) rect_out[pos] = rect_of[val];
  }
}

// ---------------------------------------------------------------------------------------
// The whole depth sort of a small frame in one workgroup: the keys stay in registers and LDS, the
// passes are as many as the keys' range needs, and a second workgroup takes the frame's totals.
// A frame of this size is a chain of launches, each mostly latency: the 12 launches of four 8-bit
// passes took 43 us at 2000 candidates, this 11 (17 at 4096). Its time grows with the keys per
// thread: 30 us at 8192, where the nine launches of three passes take 35 and hardly grow yet, so
// the line lies there.
// ---------------------------------------------------------------------------------------
constexpr int kSmallThreads = 1024;

template <int ITEMS>
__global__ __launch_bounds__(kSmallThreads) void k_depth_sort_small(const uint32_t *__restrict__ depth, uint32_t n,
                                                                    uint32_t *__restrict__ vals_out,
                                                                    const uint2 *__restrict__ rect_of,
                                                                    uint2 *__restrict__ rect_out, FrameTotals totals) {
  constexpr int WAVES = kSmallThreads / 64, DIGITS = 1 << kDepthBits, SCAN_WAVES = DIGITS / 64;
  constexpr uint32_t WTILE = 64 * ITEMS;
  __shared__ uint32_t s_keys[kSmallThreads * ITEMS], s_vals[kSmallThreads * ITEMS];
  __shared__ uint32_t s_wcnt[WAVES][DIGITS];
  __shared__ uint32_t s_red[2][WAVES], s_scan[SCAN_WAVES];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  if (blockIdx.x == 1) {
    if (tid < kBlock) frame_totals(totals);   // whole waves
    return;
  }
  uint32_t kr[ITEMS], vr[ITEMS], rr[ITEMS];
  uint32_t lo = 0xFFFFFFFFu, hi = 0u;
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const uint32_t i = (uint32_t)w * WTILE + (uint32_t)r * 64u + (uint32_t)lane;
    kr[r] = i < n ? depth[i] : kDepthNone;
    vr[r] = i;
  }
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    lo = min(lo, kr[r]);
    hi = kr[r] != kDepthNone ? max(hi, kr[r]) : hi;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    lo = min(lo, (uint32_t)__shfl_xor(lo, o, 64));
    hi = max(hi, (uint32_t)__shfl_xor(hi, o, 64));
  }
  if (lane == 0) {
    s_red[0][w] = lo;
    s_red[1][w] = hi;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < WAVES; ++k) {
    lo = min(lo, s_red[0][k]);
    hi = max(hi, s_red[1][k]);
  }
  const uint32_t range = hi > lo ? hi - lo : 0u;
  uint32_t kept = n;
  bool valid[ITEMS];
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    valid[r] = kr[r] != kDepthNone;
    kr[r] -= lo;
  }
  const unsigned long long lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  for (int shift = 0; shift == 0 || (shift < 32 && (range >> shift) != 0u); shift += kDepthBits) {
#pragma unroll
    for (int d = 0; d < DIGITS; d += 64) s_wcnt[w][d + lane] = 0u;
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
      const uint32_t d = (kr[r] >> shift) & (DIGITS - 1);
      unsigned long long peers = __ballot(valid[r]);
#pragma unroll
      for (int bit = 0; bit < kDepthBits; ++bit) {
        const bool set = (d >> bit) & 1u;
        const unsigned long long bb = __ballot(set);
        peers &= set ? bb : ~bb;
      }
      const uint32_t in_round = (uint32_t)__popcll(peers & lt);
      const uint32_t prev = s_wcnt[w][d];
      rr[r] = prev + in_round;
      if (valid[r] && in_round == 0) s_wcnt[w][d] = prev + (uint32_t)__popcll(peers);
    }
    __syncthreads();
    // thread d < DIGITS: digit d's keys before it, then per wave
    uint32_t sum = 0u, inc = 0u;
    if (w < SCAN_WAVES) {
#pragma unroll
      for (int k = 0; k < WAVES; ++k) sum += s_wcnt[k][tid];
      inc = wave_incl_scan(sum);
      if (lane == 63) s_scan[w] = inc;
    }
    __syncthreads();
    if (w < SCAN_WAVES) {
      uint32_t acc = inc - sum;
#pragma unroll
      for (int k = 0; k < SCAN_WAVES; ++k) acc += k < w ? s_scan[k] : 0u;
#pragma unroll
      for (int k = 0; k < WAVES; ++k) {
        const uint32_t c = s_wcnt[k][tid];
        s_wcnt[k][tid] = acc;
        acc += c;
      }
    }
    if (shift == 0) {
      kept = 0u;
#pragma unroll
      for (int k = 0; k < SCAN_WAVES; ++k) kept += s_scan[k];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r)
      if (valid[r]) {
        const uint32_t pos = s_wcnt[w][(kr[r] >> shift) & (DIGITS - 1)] + rr[r];
        s_keys[pos] = kr[r];
        s_vals[pos] = vr[r];
      }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
      const uint32_t i = (uint32_t)w * WTILE + (uint32_t)r * 64u + (uint32_t)lane;
      valid[r] = i < kept;
      kr[r] = valid[r] ? s_keys[i] : 0u;
      vr[r] = valid[r] ? s_vals[i] : 0u;
    }
  }
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const uint32_t i = (uint32_t)w * WTILE + (uint32_t)r * 64u + (uint32_t)lane;
    if (valid[r]) {
      vals_out[i] = vr[r];
      rect_out[i] = rect_of[vr[r]];
    }
  }
}

hipError_t launch_depth_sort_small(const DepthSort &d, int64_t n, int blocks, uint32_t *vals_out, hipStream_t s) {
  FrameTotals t = d.totals;
  t.sums = d.sums;
  t.nb = blocks;
  const auto kernel = n <= 2 * kSmallThreads ? k_depth_sort_small<2> : n <= 4 * kSmallThreads ? k_depth_sort_small<4>
                                                                                               : k_depth_sort_small<8>;
  hipLaunchKernelGGL(kernel, dim3(2), dim3(kSmallThreads), 0, s, d.keys, (uint32_t)n, vals_out, d.rect_of, d.rect_out, t);
  return hipGetLastError();
}

// Keys per thread from the sort's capacity.
int radix_items(int64_t n_max) {
  return n_max >= kRadixHugeSort ? kSortItemsHuge : n_max >= kRadixBigSort ? kSortItemsBig : kSortItems;
}

static int64_t radix_stride(int64_t n_max) {
  const int64_t tile = (int64_t)kBlock * radix_items(n_max);
  return ((n_max + tile - 1) / tile + 7) & ~(int64_t)7;
}

size_t radix_hist_bytes(int64_t n_max, bool depth) {
  return 4 * (size_t)(depth ? kDepthRadix : kRadix) * (size_t)radix_stride(n_max);
}

static FrameTotals first_totals(const DepthSort &d, int blocks) {
  FrameTotals t = d.totals;
  t.sums = d.part;
  t.nb = blocks;
  return t;
}

// Sort (keys, vals) by the low `bits` bits of the keys; stable. Ping-pongs between
// buffers [0] and [1]; *result_buf receives the index holding the result. hist and scan
// hold radix_hist_bytes(n_max) each (16-byte aligned). `depth`: see DepthSort.
template <int RB, int ITEMS>
static void radix_passes(uint32_t *keys[2], uint32_t *vals[2], uint32_t *n_ptr, int64_t n_max, int bits,
                         uint32_t *hist, uint32_t *scan, uint32_t *tot, int *cur_out, const DepthSort *depth,
                         hipStream_t s) {
  constexpr int TILE = kBlock * ITEMS;
  const int nb_max = (int)((n_max + TILE - 1) / TILE);
  const int stride = (int)radix_stride(n_max);
  const uint32_t n_all = (uint32_t)n_max;
  const unsigned grid = xcd_grid(nb_max);
  int cur = 0;
  // the fewest passes of at most RB digit bits, the bits spread evenly over them
  const int passes = (bits + RB - 1) / RB;
  for (int pass = 0, shift = 0; pass < passes; ++pass) {
    const int nbits = bits / passes + (pass < bits % passes ? 1 : 0);
    const uint32_t dmask = (1u << nbits) - 1u;
    const bool first = pass == 0 && depth;
    const bool last = pass == passes - 1 && depth;
    const uint32_t *kin = first ? depth->keys : keys[cur];
    if (first)
      hipLaunchKernelGGL(HIP_KERNEL_NAME(k_rs_hist<RB, ITEMS, true>), dim3(grid), dim3(kBlock), 0, s, kin, n_ptr, n_all,
                         shift, dmask, hist, stride, depth->sums, depth->part);
    else
      hipLaunchKernelGGL(HIP_KERNEL_NAME(k_rs_hist<RB, ITEMS, false>), dim3(grid), dim3(kBlock), 0, s, kin, n_ptr, n_all,
                         shift, dmask, hist, stride, nullptr, nullptr);
    // the first pass's workgroups cover all candidates; the later passes' the count it kept
    if (first)
      hipLaunchKernelGGL(k_rs_scan<true>, dim3((1 << RB) + 1), dim3(kBlock), 0, s, nullptr, n_all, hist, scan, tot,
                         stride, TILE, first_totals(*depth, nb_max));
    else
      hipLaunchKernelGGL(k_rs_scan<false>, dim3(1 << RB), dim3(kBlock), 0, s, n_ptr, n_all, hist, scan, tot, stride, TILE,
                         FrameTotals{});
    const uint2 *rect_of = last ? depth->rect_of : nullptr;
    uint2 *rect_out = last ? depth->rect_out : nullptr;
    auto kernel = first ? k_rs_scatter<RB, ITEMS, false, true> : last ? k_rs_scatter<RB, ITEMS, true, false>
                                                                      : k_rs_scatter<RB, ITEMS, false, false>;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(kBlock), 0, s, kin, vals[cur], keys[cur ^ 1], vals[cur ^ 1], n_ptr,
                       n_all, n_ptr, shift, dmask, hist, scan, tot, stride, rect_of, rect_out);
    cur ^= 1;
    shift += nbits;
  }
  *cur_out = cur;
}

hipError_t launch_radix_sort(uint32_t *keys[2], uint32_t *vals[2], uint32_t *n_ptr, int64_t n_max,
                             int bits, uint32_t *hist, uint32_t *scan, uint32_t *tot, int *result_buf,
                             hipStream_t s, const DepthSort *depth) {
  *result_buf = 0;
  if (depth) bits = depth->far ? kDepthFarBits : 3 * kDepthBits;
  if (n_max <= 0) return hipSuccess;
  const auto run = [&](auto items) {
    constexpr int I = decltype(items)::value;
    // nine-bit digits where that makes a pass fewer
    if (depth ? !depth->far : (bits + kDepthBits - 1) / kDepthBits < (bits + kRadixBits - 1) / kRadixBits)
      radix_passes<kDepthBits, I>(keys, vals, n_ptr, n_max, bits, hist, scan, tot, result_buf, depth, s);
    else
      radix_passes<kRadixBits, I>(keys, vals, n_ptr, n_max, bits, hist, scan, tot, result_buf, depth, s);
  };
  switch (radix_items(n_max)) {
    case kSortItemsHuge: run(std::integral_constant<int, kSortItemsHuge>{}); break;
    case kSortItemsBig: run(std::integral_constant<int, kSortItemsBig>{}); break;
    default: run(std::integral_constant<int, kSortItems>{}); break;
  }
  return hipGetLastError();
}

hipError_t launch_row_scan(const uint32_t *n_ptr, const uint32_t *hist, uint32_t *scan, uint32_t *tot, int rows,
                           int stride, int tile, hipStream_t s) {
  hipLaunchKernelGGL(k_rs_scan<false>, dim3((unsigned)rows), dim3(kBlock), 0, s, n_ptr, 0u, hist, scan, tot, stride,
                     tile, FrameTotals{});
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Bucket ranges from the sorted bucket ids (ranges zeroed beforehand); the id count is read on
// the device, the grid covers k_max ids.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_ranges(const uint32_t *__restrict__ ids, int shift, const uint32_t *k_ptr,
                                                   uint2 *__restrict__ ranges) {
  const uint32_t K = *k_ptr;
  const uint32_t k0 = 4u * (blockIdx.x * kBlock + threadIdx.x);   // four ids per thread
  if (k0 >= K) return;
  uint32_t t[4];
  if (k0 + 4u <= K) {
    const uint4 v = *reinterpret_cast<const uint4 *>(ids + k0);
    t[0] = v.x; t[1] = v.y; t[2] = v.z; t[3] = v.w;
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) t[i] = (k0 + i < K) ? ids[k0 + i] : 0u;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) t[i] >>= shift;
  uint32_t prev = (k0 > 0u) ? ids[k0 - 1u] >> shift : 0xFFFFFFFFu;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t k = k0 + i;
    if (k >= K) break;
    if (t[i] != prev) {
      ranges[t[i]].x = k;
      if (k > 0u) ranges[prev].y = k;
    }
    prev = t[i];
  }
  if (k0 + 4u >= K) ranges[prev].y = K;   // the last id closes its bucket
}

// 16-byte stores over the aligned body (grid-stride), single words before and after it.
__global__ __launch_bounds__(kBlock) void k_fill_u32(uint32_t *p, uint32_t v, int64_t n) {
  const int64_t lead = min(n, (int64_t)(((16u - (uint32_t)(reinterpret_cast<uintptr_t>(p) & 15u)) & 15u) / 4u));
  const int64_t n4 = (n - lead) / 4;
  uint4 *q = reinterpret_cast<uint4 *>(p + lead);
  const uint4 vv = make_uint4(v, v, v, v);
  const int64_t stride = (int64_t)gridDim.x * kBlock;
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n4; i += stride) q[i] = vv;
  if (blockIdx.x == 0) {
    const int64_t tail = lead + 4 * n4;
    if ((int64_t)threadIdx.x < lead) p[threadIdx.x] = v;
    if ((int64_t)threadIdx.x < n - tail) p[tail + threadIdx.x] = v;
  }
}

hipError_t launch_fill_u32(uint32_t *p, uint32_t v, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t groups = (n / 4 + kBlock - 1) / kBlock;
  const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>(groups, 4096));
  hipLaunchKernelGGL(k_fill_u32, dim3(grid), dim3(kBlock), 0, s, p, v, n);
  return hipGetLastError();
}

hipError_t launch_ranges(const uint32_t *ids, int shift, const uint32_t *k_ptr, int64_t k_max, uint2 *ranges,
                         hipStream_t s) {
  if (k_max <= 0) return hipSuccess;
  const int64_t threads = (k_max + 3) / 4;
  hipLaunchKernelGGL(k_ranges, dim3((unsigned)((threads + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, ids, shift,
                     k_ptr, ranges);
  return hipGetLastError();
}

}  // namespace flod
