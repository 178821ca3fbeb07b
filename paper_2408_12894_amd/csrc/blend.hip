// Front-to-back alpha compositing (Preliminary section: eq. 2 and blending in depth order).
//
// One workgroup per 16x16 tile, one pixel per thread. The tile's
// sorted list is consumed in batches of 256 entries (48 bytes each in LDS: mu' and its
// residual, conic, opacity, colour, decoded once per entry). Per pixel:
//   q = d^T conic d (d = pixel centre - mu', mu' = hi + lo); skip if q > 9 (evaluated as
//   k q in the completed-square form of conic_stage, k the scale of exp2)
//   alpha = min(0.99, o exp(-q/2)); skip if alpha < 1/255
//   stop (without blending) once T (1 - alpha) < 1e-4
//   C += alpha T c; T *= 1 - alpha
// T and the colours are FP32: T takes one rounding per blended contributor, so after m of
// them its relative error grows like sqrt(m) ulp (about 2e-6 at a thousand), far inside the
// relative 1e-4 margin around the stop threshold that the parity checks flag.
// The workgroup leaves the list as soon as all 256 pixels have stopped.
//
// Workgroups take the tiles in order of decreasing list length (see tile_order). Each tile also
// lists the entries it blended into some pixel, the only ones its backward pass processes:
// (list position, Gaussian) pairs in list order at the start of the tile's range, and their
// count, from which the backward orders its tiles.
#include <type_traits>

#include "blend_common.h"

namespace flod {

// Appends the entries of the staged batch at list position bstart that some pixel blended
// (s_taken) to the tile's list of blended entries (out, n_bl entries so far; the count is the
// same in every thread). Called by every thread of the workgroup after a barrier that follows
// the batch's walk; thread t handles the entries t, t + NT, ...
template <int NT>
__device__ __forceinline__ void append_blended(const uint8_t *s_taken, const uint32_t *s_id, uint32_t *s_wcnt,
                                               int bstart, int n, uint2 *out, uint32_t &n_bl, int tid) {
  constexpr int W = NT / 64;
  const int lane = tid & 63, w = tid >> 6;
  const unsigned long long below = lane ? (~0ull >> (64 - lane)) : 0ull;
  for (int e0 = 0; e0 < kBatch; e0 += NT) {
    const int e = e0 + tid;
    const bool f = bstart + e < n && s_taken[e] != 0;
    const unsigned long long m = __ballot(f);
    if (lane == 0) s_wcnt[w] = (uint32_t)__popcll(m);
    __syncthreads();
    uint32_t off = n_bl, tot = 0;
#pragma unroll
    for (int v = 0; v < W; ++v) {
      const uint32_t c = s_wcnt[v];
      off += v < w ? c : 0u;
      tot += c;
    }
    if (f) out[off + (uint32_t)__popcll(m & below)] = make_uint2((uint32_t)(bstart + e), s_id[e]);
    n_bl += tot;
    if (e0 + NT < kBatch) __syncthreads();   // s_wcnt is written again
  }
}

template <int CTRL>
__device__ __forceinline__ uint32_t or_dpp(uint32_t v) {
  return v | (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}

// The OR of a value over the wave's 64 lanes.
__device__ __forceinline__ uint32_t wave_or(uint32_t v) {
  v = or_dpp<0x121>(or_dpp<0x122>(or_dpp<0x124>(or_dpp<0x128>(v))));   // over each row of 16 (rotations)
  uint32_t x = 0u;
#pragma unroll
  for (int r = 0; r < 4; ++r) x |= (uint32_t)__builtin_amdgcn_readlane((int)v, 16 * r);
  return x;
}

// The list is walked in groups of U entries: their l first (independent of each other and of the
// pixel's state, their LDS reads in flight together), then the entries in turn. Two ways to
// take the entries:
//  - branches (PRED false): a pixel that the entry does not reach skips its arithmetic. A wave
//    issues least where few of its pixels are reached.
//  - predicated (PRED true): every entry's arithmetic runs with alpha 0 where it does not
//    reach the pixel, without a branch: two VALU more for a pixel reached, but no exec-mask and
//    branch latency between the entries, which is what a walk takes where the device has few
//    waves per SIMD, and the better way too where footprints are large.
// Both make the same operations in the same order on what a pixel blends. A pixel that stopped
// has T kept and Tw = 0, so that further weights are 0. A weight of 0 may not meet a colour that
// is not finite: batches that hold one select the sums instead.
//
// Groups (k_blend per frame, us): one entry at a time with branches, as it was; U = 4 branches;
// U = 4, 8, 16 predicated
//   2k at 128x128, 64 tiles              42.4 | 39.6 |   -   33.1  28.3
//   levels 1-2 at 640x360, 920 tiles    153.5 | 142.6 |   -  107.3  95.4
//   500k at 1280x720, 3,600 tiles        81.5 |  78.8 |  84.4  76.4  72.2
//   1M at 1920x1080, 8,160 tiles        127.7 | 123.0 | 138.2 132.0 142.9
//   levels 1-5 at 1920x1080             125.7 | 121.7 | 111.7 108.5 117.5
//   2.5M (floor 0.0125) at 3840x2160    357.2 | 345.4 | 329.6 339.1 392.5
// U = 16 takes 125 registers (four waves per SIMD), U = 8 78, branches with U = 4 64 (eight
// waves); branches with U = 8 or 16 hold the group's colours in registers to no use (154, 254 us
// at 1M). Skipping an entry that no pixel of the wave takes cost as much as it saved.
//
// COUNT: the caller wants each pixel's count of blended entries (n_blended).
template <int U, bool PRED, bool COUNT>
__global__ __launch_bounds__(kTile * kTile) void k_blend(const uint2 *__restrict__ ranges,
                                                         const uint32_t *__restrict__ values,
                                                         const float4 *__restrict__ xyab,
                                                         const float4 *__restrict__ cop,
                                                         const float2 *__restrict__ blue, int W, int H, int tiles_x,
                                                         float bg0, float bg1, float bg2, float *__restrict__ image,
                                                         float *__restrict__ final_T, int32_t *__restrict__ n_contrib,
                                                         int32_t *__restrict__ n_blended, uint2 *__restrict__ blended,
                                                         uint32_t *__restrict__ tile_blended,
                                                         const uint32_t *__restrict__ order) {
  constexpr int NT = kTile * kTile;
  static_assert(kBatch == NT && kBatch % U == 0, "one staged entry per thread, whole groups");
  __shared__ float4 s_a[kBatch];
  __shared__ float4 s_b[kBatch];
  __shared__ float4 s_c[kBatch];
  __shared__ uint8_t s_taken[kBatch];
  __shared__ uint32_t s_id[kBatch];
  __shared__ uint32_t s_wcnt[NT / 64];
  const int tile = (int)order[blockIdx.x];
  const int tid = threadIdx.x, lane = tid & 63;
  const int x0 = (tile % tiles_x) * kTile, y0 = (tile / tiles_x) * kTile;
  const int px = x0 + (tid & (kTile - 1)), py = y0 + (tid >> 4);
  // pixel centres relative to the tile's corner
  const float fx = (float)(tid & (kTile - 1)) + 0.5f, fy = (float)(tid >> 4) + 0.5f;
  const bool inside = px < W && py < H;
  float T = 1.0f, C0 = 0.0f, C1 = 0.0f, C2 = 0.0f;
  int last = 0, nbl = 0;
  bool done = !inside;
  float Tw = inside ? 1.0f : 0.0f;   // PRED: T while the pixel is blending, then 0
  const uint2 rg = ranges[tile];
  const int n = (int)(rg.y - rg.x);
  int last_start = -1;   // start of the last batch walked
  uint32_t n_bl = 0;     // blended entries listed so far
  for (int start = 0; start < n; start += kBatch) {
    if (__syncthreads_and(done)) break;
    // the previous batch's blended entries join the list, this batch's flags start at zero
    if (blended && start > 0)
      append_blended<NT>(s_taken, s_id, s_wcnt, start - kBatch, n, blended + rg.x, n_bl, tid);
    s_taken[tid] = 0;
    if (start + tid < n) {
      const uint32_t g = values[rg.x + start + tid];
      s_id[tid] = g;
      stage_entry(xyab, cop, blue, g, x0, y0, s_a[tid], s_b[tid], s_c[tid]);
    } else if (start + tid < n + U) {
      // past the list up to a whole group: entries that no pixel takes
      s_a[tid] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      s_b[tid] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      s_c[tid] = make_float4(INFINITY, 0.0f, 0.0f, 0.0f);
    }
    bool finite = true;   // PRED: every staged colour is
    if (PRED)
      finite = __syncthreads_and(start + tid >= n ||
                                 (isfinite(s_b[tid].z) && isfinite(s_b[tid].w) && isfinite(s_c[tid].y)));
    else
      __syncthreads();
    // the count is the same in every lane (read from the first: the loop's exit test is then a
    // scalar compare instead of a VALU one per entry)
    const int cnt = __builtin_amdgcn_readfirstlane(min(kBatch, n - start));
    for (int j0 = 0; j0 < cnt; j0 += U) {
      if (!__any(PRED ? Tw != 0.0f : !done)) break;
      float l[U], thr[U], c0[U], c1[U], c2[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float4 A = s_a[j0 + u];
        const float4 B = s_b[j0 + u];
        const float2 BL = *reinterpret_cast<const float2 *>(&s_c[j0 + u]);   // threshold on l, blue
        const float dx = fx - A.x;
        const float t = conic_column(A.w, dx, B.y);
        l[u] = conic_kq(B.x, A.z, dx, fy - A.y, t);   // k q + log2 o
        thr[u] = BL.x;
        c0[u] = B.z;
        c1[u] = B.w;
        c2[u] = BL.y;
      }
      if (PRED) {
        float al[U];   // alpha, 0 where the entry does not reach the pixel
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const float a = fminf(kAlphaMax, alpha_from_log2(l[u]));
          al[u] = l[u] < thr[u] ? 0.0f : a;
        }
        uint32_t bits = 0u;   // the pixel's taken entries, the last one in bit 0
        auto walk = [&](auto finite) {
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const float Tn = fmaf(-al[u], Tw, Tw);
            const bool stop = Tn < kTMin;                // also once Tw is 0
            const float wgt = stop ? 0.0f : al[u] * Tw;
            const bool take = wgt > 0.0f;
            Tw = stop ? 0.0f : Tn;
            T = stop ? T : Tn;
            if (decltype(finite)::value) {
              C0 = fmaf(wgt, c0[u], C0);
              C1 = fmaf(wgt, c1[u], C1);
              C2 = fmaf(wgt, c2[u], C2);
            } else {
              C0 = take ? fmaf(wgt, c0[u], C0) : C0;
              C1 = take ? fmaf(wgt, c1[u], C1) : C1;
              C2 = take ? fmaf(wgt, c2[u], C2) : C2;
            }
            bits = bits + bits + (take ? 1u : 0u);
          }
        };
        if (finite)
          walk(std::true_type{});
        else
          walk(std::false_type{});
        if (bits) last = start + j0 + U + 1 - __ffs((int)bits);
        if (COUNT) nbl += __popc(bits);
        if (blended) {
          const uint32_t any = wave_or(bits);
          if (lane < U && ((any >> (U - 1 - lane)) & 1u)) s_taken[j0 + lane] = 1;
        }
        done = Tw == 0.0f;
      } else
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (done || l[u] < thr[u]) continue;                      // q > 9 or alpha < 1/255
        const float alpha = fminf(kAlphaMax, alpha_from_log2(l[u]));
        const float wgt = alpha * T;
        const float Tn = fmaf(-alpha, T, T);   // T (1 - alpha), one rounding
        if (Tn < kTMin) {
          done = true;
          continue;
        }
        C0 = fmaf(wgt, c0[u], C0);
        C1 = fmaf(wgt, c1[u], C1);
        C2 = fmaf(wgt, c2[u], C2);
        T = Tn;
        last = start + j0 + u + 1;
        if (COUNT) ++nbl;
        s_taken[j0 + u] = 1;
      }
    }
    last_start = start;
  }
  // the blended entries of the last batch walked (the walk blends nothing after it)
  __syncthreads();
  if (blended && last_start >= 0)
    append_blended<NT>(s_taken, s_id, s_wcnt, last_start, n, blended + rg.x, n_bl, tid);
  if (tid == 0 && tile_blended) tile_blended[tile] = n_bl;
  if (!inside) return;
  const size_t plane = (size_t)W * H, pix = (size_t)py * W + px;
  image[pix] = fmaf(T, bg0, C0);
  image[plane + pix] = fmaf(T, bg1, C1);
  image[2 * plane + pix] = fmaf(T, bg2, C2);
  final_T[pix] = T;
  n_contrib[pix] = last;
  if (COUNT) n_blended[pix] = nbl;
}

constexpr int kFewTiles = 4096;

hipError_t launch_blend(const uint2 *ranges, const uint32_t *values, const float4 *xyab, const float4 *cop,
                        const float2 *blue, const DevCamera &cam, const float bg[3], float *image, float *final_T,
                        int32_t *n_contrib, int32_t *n_blended, uint2 *blended, uint32_t *tile_blended,
                        const uint32_t *order, bool large, hipStream_t s) {
  const int n_tiles = cam.tiles_x * cam.tiles_y;
  // 16 predicated entries per group while the frame has few waves for the device; beyond, eight
  // where the levels' scale floors make footprints large, else branches (see the table)
  const int way = n_tiles <= kFewTiles ? 0 : large ? 1 : 2;
  auto kernel = way == 0 ? n_blended ? k_blend<16, true, true> : k_blend<16, true, false>
                : way == 1 ? n_blended ? k_blend<8, true, true> : k_blend<8, true, false>
                           : n_blended ? k_blend<4, false, true> : k_blend<4, false, false>;
  hipLaunchKernelGGL(kernel, dim3(n_tiles), dim3(kTile * kTile), 0, s, ranges, values, xyab, cop, blue, cam.W, cam.H,
                     cam.tiles_x, bg[0], bg[1], bg[2], image, final_T, n_contrib, n_blended, blended, tile_blended,
                     order);
  return hipGetLastError();
}

}  // namespace flod
