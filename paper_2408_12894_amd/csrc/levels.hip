// Whole-level operations on the resident stack.
//
// Compaction keeps a subset of a level's Gaussians, in index order, in caller-provided
// arrays. The subset is either the eq. 6 band around a fixed centre (the predetermined
// selection set, section Selective Rendering: rendering the compacted levels together gives
// the same image as selective rendering around that centre, while only the kept Gaussians
// stay resident and can be stored) or a per-Gaussian keep mask (overlap pruning, section
// Overlap Pruning). Two passes: per-workgroup counts, then (after a scan) a copy of the
// kept Gaussians' 59 attributes (236 bytes), whose output rows are consecutive: a workgroup
// lists its kept Gaussians and copies each array's rows as one run, thread by thread in
// output order.
//
// The level transition (section Training Method, eq. 5) clones a trained level into the
// initial state of the next one with s_opt = log(s^(l) - s_min^(l+1)), so that the next
// level's eq. 4 scale starts equal to s^(l).
#include "project.h"

namespace flod {

struct BandKeep {
  const float *means;
  float c[3];
  float lo2, hi2;
  __device__ __forceinline__ bool operator()(int64_t i) const {
    const float d2 = dist2(means[i * 3 + 0], means[i * 3 + 1], means[i * 3 + 2], c);
    return (lo2 <= d2) && (d2 < hi2);
  }
};

struct MaskKeep {
  const uint8_t *mask;
  __device__ __forceinline__ bool operator()(int64_t i) const { return mask[i] != 0; }
};

__global__ __launch_bounds__(kBlock) void k_mask_count(MaskKeep keep_of, int64_t n, uint32_t *block_cnt) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const bool keep = (i < n) && keep_of(i);
  const int cnt = __syncthreads_count(keep);
  if (threadIdx.x == 0) block_cnt[blockIdx.x] = (uint32_t)cnt;
}

// The counts of all levels' bands in one launch (three levels' counts and scans in six launches
// took 36 us for 4.2M Gaussians, in two they take 25).
__global__ __launch_bounds__(kBlock) void k_band_count(BandCounts c, uint32_t *block_cnt) {
  int l = 0;
  while (l + 1 < c.levels && (int64_t)blockIdx.x >= c.first[l + 1]) ++l;
  const int64_t i = ((int64_t)blockIdx.x - c.first[l]) * kBlock + threadIdx.x;
  const BandKeep keep_of{c.means[l], {c.centre[0], c.centre[1], c.centre[2]}, c.lo2[l], c.hi2[l]};
  const int cnt = __syncthreads_count(i < c.n[l] && keep_of(i));
  if (threadIdx.x == 0) block_cnt[blockIdx.x] = (uint32_t)cnt;
}

// One array's rows of the kept Gaussians: W values of type T per row, output rows consecutive.
// U values per thread are loaded together.
template <int W, class T>
__device__ __forceinline__ void copy_rows(const T *__restrict__ src, T *__restrict__ dst, const uint8_t *s_src, int kept) {
  constexpr int U = 4;
  const int n = kept * W;
  for (int f0 = threadIdx.x; f0 < n; f0 += U * kBlock) {
    T v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int f = min(f0 + u * kBlock, n - 1);
      v[u] = src[(int)s_src[f / W] * W + f % W];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (f0 + u * kBlock < n) dst[f0 + u * kBlock] = v[u];
  }
}

// Bound by HBM: one Gaussian per thread, its 192-byte SH row in 12 loads and stores that each
// touched 64 cache lines, 2.18M of 4.2M Gaussians took 634 us (1.6 TB/s); now 224 us (4.6 TB/s).
template <class Keep>
__global__ __launch_bounds__(kBlock) void k_keep_copy(Keep keep_of, flod_level in,
                                                      const unsigned long long *prefix, flod_level out) {
  __shared__ uint32_t s_w[kBlock / 64];
  __shared__ uint8_t s_src[kBlock];
  const int64_t base = (int64_t)blockIdx.x * kBlock, i = base + threadIdx.x;
  const bool keep = (i < in.n) && keep_of(i);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const unsigned long long m = __ballot(keep);
  if (lane == 0) s_w[w] = (uint32_t)__popcll(m);
  __syncthreads();
  uint32_t at = 0, kept = 0;
#pragma unroll
  for (int k = 0; k < kBlock / 64; ++k) {
    at += k < w ? s_w[k] : 0u;
    kept += s_w[k];
  }
  if (keep) s_src[at + (uint32_t)__popcll(m & (lane ? ~0ull >> (64 - lane) : 0ull))] = (uint8_t)threadIdx.x;
  __syncthreads();
  const int64_t o = (int64_t)prefix[blockIdx.x];
  constexpr int kRow4 = FLOD_SH_COEFFS * 3 / 4;
  copy_rows<kRow4>(reinterpret_cast<const float4 *>(in.sh) + base * kRow4,
                   reinterpret_cast<float4 *>(const_cast<float *>(out.sh)) + o * kRow4, s_src, (int)kept);
  copy_rows<1>(reinterpret_cast<const float4 *>(in.quats) + base,
               reinterpret_cast<float4 *>(const_cast<float *>(out.quats)) + o, s_src, (int)kept);
  copy_rows<3>(in.means + base * 3, const_cast<float *>(out.means) + o * 3, s_src, (int)kept);
  copy_rows<3>(in.log_scales + base * 3, const_cast<float *>(out.log_scales) + o * 3, s_src, (int)kept);
  copy_rows<1>(in.opacity_logits + base, const_cast<float *>(out.opacity_logits) + o, s_src, (int)kept);
}

static unsigned grid_of(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

hipError_t launch_select_count(const BandCounts &c, uint32_t *block_cnt, hipStream_t s) {
  const int64_t blocks = c.first[c.levels];
  if (blocks <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_band_count, dim3((unsigned)blocks), dim3(kBlock), 0, s, c, block_cnt);
  return hipGetLastError();
}

hipError_t launch_select_copy(const flod_level &in, const float centre[3], float lo2, float hi2,
                              const unsigned long long *prefix, const flod_level &out, hipStream_t s) {
  if (in.n <= 0) return hipSuccess;
  const BandKeep k{in.means, {centre[0], centre[1], centre[2]}, lo2, hi2};
  hipLaunchKernelGGL(k_keep_copy<BandKeep>, dim3(grid_of(in.n)), dim3(kBlock), 0, s, k, in, prefix, out);
  return hipGetLastError();
}

hipError_t launch_mask_count(const uint8_t *mask, int64_t n, uint32_t *block_cnt, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_mask_count, dim3(grid_of(n)), dim3(kBlock), 0, s, MaskKeep{mask}, n, block_cnt);
  return hipGetLastError();
}

hipError_t launch_mask_copy(const flod_level &in, const uint8_t *mask, const unsigned long long *prefix,
                            const flod_level &out, hipStream_t s) {
  if (in.n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_keep_copy<MaskKeep>, dim3(grid_of(in.n)), dim3(kBlock), 0, s, MaskKeep{mask}, in, prefix,
                     out);
  return hipGetLastError();
}

// eq. 5 over the level's five arrays as consecutive segments of float4 slots, one slot per
// thread: log_scales transformed, the others copied (those the output shares with the input, in
// an in-place transition, have no slots). s^(l) is formed as the rasterizer's eq. 4 forms it
// (exp in FP64 rounded once to FP32, plus s_min^(l) in FP64); the logarithm is FP64, rounded to
// FP32. Bound by HBM (472 B per Gaussian); one thread per Gaussian, each SH row in 12 loads and
// stores that each touched 64 cache lines, took 343 us for 1.2M Gaussians (1.7 TB/s); now 114 us (5.0 TB/s).
struct TransitionSeg {
  const float *src;
  float *dst;
  int64_t len;      // floats
  int64_t first4;   // first float4 slot
  int vec;          // both 16-byte aligned
};

struct TransitionArgs {
  TransitionSeg seg[5];   // log_scales, means, quats, opacity logits, SH
  int64_t total4;
  double s_min_l, s_min_next;
};

__device__ __forceinline__ float next_scale(float v, const TransitionArgs &a) {
  return (float)log(((double)exp_rn1(v) + a.s_min_l) - a.s_min_next);
}

__global__ __launch_bounds__(kBlock) void k_level_transition(TransitionArgs a) {
  const int64_t q = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (q >= a.total4) return;
  TransitionSeg S = a.seg[0];
  int s = 0;
#pragma unroll
  for (int k = 1; k < 5; ++k)
    if (q >= a.seg[k].first4) {
      S = a.seg[k];
      s = k;
    }
  const int64_t e = (q - S.first4) * 4;
  if (S.vec && e + 4 <= S.len) {
    float4 v = *reinterpret_cast<const float4 *>(S.src + e);
    if (s == 0) v = make_float4(next_scale(v.x, a), next_scale(v.y, a), next_scale(v.z, a), next_scale(v.w, a));
    *reinterpret_cast<float4 *>(S.dst + e) = v;
    return;
  }
  for (int64_t c = e; c < e + 4 && c < S.len; ++c) S.dst[c] = s == 0 ? next_scale(S.src[c], a) : S.src[c];
}

hipError_t launch_level_transition(const flod_level &in, float s_min_next, const flod_level &out, hipStream_t s) {
  if (in.n <= 0) return hipSuccess;
  const float *src[5] = {in.log_scales, in.means, in.quats, in.opacity_logits, in.sh};
  const float *dst[5] = {out.log_scales, out.means, out.quats, out.opacity_logits, out.sh};
  const int64_t width[5] = {3, 3, 4, 1, FLOD_SH_COEFFS * 3};
  TransitionArgs a;
  a.s_min_l = (double)in.s_min;
  a.s_min_next = (double)s_min_next;
  int64_t slot = 0;
  for (int k = 0; k < 5; ++k) {
    TransitionSeg &S = a.seg[k];
    S.src = src[k];
    S.dst = const_cast<float *>(dst[k]);
    S.len = k > 0 && src[k] == dst[k] ? 0 : in.n * width[k];
    S.first4 = slot;
    S.vec = reinterpret_cast<uintptr_t>(src[k]) % 16 == 0 && reinterpret_cast<uintptr_t>(dst[k]) % 16 == 0;
    slot += (S.len + 3) / 4;
  }
  a.total4 = slot;
  hipLaunchKernelGGL(k_level_transition, dim3((unsigned)((slot + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, a);
  return hipGetLastError();
}

}  // namespace flod
