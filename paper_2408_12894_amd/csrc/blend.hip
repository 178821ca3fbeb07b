// Front-to-back alpha compositing (Preliminary section: eq. 2 and blending in depth order).
//
// One workgroup per 16x16 tile, one pixel per thread, one quadrant of 8x8 pixels per wave. The
// tile's sorted list is consumed in batches of 256 entries (48 bytes each in LDS: mu' and its
// residual, conic, opacity, colour, decoded once per entry), of which each wave walks those
// that may reach its quadrant (reach_mask). Per pixel:
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

// The quadrants (8 x 8 pixels, bit = column + 2 row) of its tile that a staged entry may reach: those
// whose box of pixel centres meets the ellipse P = l2o - thr, P = E dx^2 + C (dy + r dx)^2 = -k q. The
// least P over the box lies on the side nearest the mean in x or the one nearest in y. The walk's
// own P of a pixel, in FP32 from the same staged values, is off by a few ulp and by what the
// rounding of dy + r dx makes, at most 2^-22 M of its terms' size M: its root is then at least the
// root of the least P, less sqrt(C) 2^-22 M. The margins are four times that, 1e-5 in P and a
// relative 1e-5, and only a comparison that holds drops a quadrant (so none for NaN).
__device__ __forceinline__ uint32_t reach_mask(const float4 &a, const float4 &b, float thr) {
  const float E = -a.w, C = -b.x, r = a.z;
  if (!(E > 0.0f && C > 0.0f)) return 15u;
  const float xl = 0.5f - a.x, yl = 0.5f - a.y;
  const float M = fabsf(r) * fmaxf(fabsf(xl), fabsf(xl + 15.0f)) + fmaxf(fabsf(yl), fabsf(yl + 15.0f));
  float lim = sqrtf(fmaxf(b.y - thr, 0.0f) + 1e-5f) + 0x1p-20f * sqrtf(C) * M;
  lim = lim * lim * 1.00001f;
  const float g = -C * r * __builtin_amdgcn_rcpf(fmaf(C * r, r, E));   // the least P of a row lies at dx = g dy
  uint32_t mask = 0u;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float xa = xl + 8.0f * (float)(q & 1), ya = yl + 8.0f * (float)(q >> 1);
    const float xe = fminf(fmaxf(0.0f, xa), xa + 7.0f), ye = fminf(fmaxf(0.0f, ya), ya + 7.0f);
    const float y1 = fminf(fmaxf(-r * xe, ya), ya + 7.0f), x2 = fminf(fmaxf(g * ye, xa), xa + 7.0f);
    const float v1 = fmaf(r, xe, y1), v2 = fmaf(r, x2, ye);
    const float P1 = fmaf(E * xe, xe, C * v1 * v1), P2 = fmaf(E * x2, x2, C * v2 * v2);
    if (!(P1 > lim && P2 > lim)) mask |= 1u << q;
  }
  return mask;
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
//    waves per SIMD. Listing the blended entries costs it a wave-wide OR per group besides.
// Both make the same operations in the same order on what a pixel blends. A pixel that stopped
// has T kept and Tw = 0, so that further weights are 0. A weight of 0 may not meet a colour that
// is not finite: batches that hold one select the sums instead.
//
// Groups (k_blend per frame, us): one entry at a time with branches over the whole list, as it was;
// then over the entries that reach the wave's quadrant, U = 4 branches; U = 4, 8, 16 predicated
//   2k at 128x128, 64 tiles              42.4 |   -   |  21.4  18.3  19.2
//   levels 1-2 at 640x360, 920 tiles    153.5 |   -   | 101.0  89.5  96.2
//   500k at 1280x720, 3,600 tiles        81.5 |   -   |  64.8  60.8  64.4
//   1M at 1920x1080, 8,160 tiles        127.7 | 107.7 | 111.2 117.0    -
//   levels 1-5 at 1920x1080             125.7 | 116.4 | 104.4 105.6 123.2
//   2.5M (floor 0.0125) at 3840x2160    357.2 | 349.5 | 331.1 360.2 422.9
// Over the whole list the best were 28.3 (U = 16), 95.4 (16), 72.2 (16), 123.0 (branches), 108.5 (8)
// and 329.6 us (4): what a quadrant's list leaves out is a third of the entries where footprints
// are a few tiles, a tenth where they are many. The more entries a group, the more registers it
// holds (U = 16 four waves per SIMD). Branches with U = 8 or 16 hold the group's colours in
// registers to no use (154, 254 us at 1M), U = 2 waits more often (116).
//
// AHEAD: each group is read, and its alphas found, before the one in front of it is taken. Where a
// SIMD has few waves none of them covers another's LDS reads; the two groups' registers (167) cost
// nothing there. us per kernel, without and with: 2k at 253x187 (192 tiles) 12.1 11.7, 20k at 400x300
// (475) 36.7 32.8, levels 1-2 at 640x360 (920) 88.9 80.8, 100k at 800x600 (1,900) 65.4 60.1, 300k
// clusters at 1000x700 (2,772) 108 105, 500k clusters at 1280x720 (3,600) 127 129 and, floor 0.0125,
// 62 69; U = 4 ahead 19.7 and 88.9 at 2k / 128x128 and levels 1-2, against 17.5 and 80.8. A walk of
// several waves per quadrant, the alphas found by one or two and blended by another, took 17.1
// and 88.4 at best there.
//
// COUNT: the caller wants each pixel's count of blended entries (n_blended).
template <int U, bool PRED, bool AHEAD, bool COUNT>
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
  static_assert(PRED || !AHEAD, "ahead: the predicated way only");
  constexpr int kFill = AHEAD ? 2 * U : U;   // places filled behind a wave's entries
  constexpr int W4 = NT / 64;
  // the staged entries, and behind them one that no pixel takes
  __shared__ float4 s_a[kBatch + 1];
  __shared__ float4 s_b[kBatch + 1];
  __shared__ float4 s_c[kBatch + 1];
  __shared__ __align__(16) uint16_t s_off[W4][kBatch + kFill];   // each wave's entries: byte offsets into s_a
  __shared__ uint8_t s_reach[kBatch];                        // the waves each entry may reach
  __shared__ uint8_t s_taken[kBatch];
  __shared__ uint32_t s_id[kBatch];
  __shared__ uint32_t s_wcnt[NT / 64];
  const int tile = (int)order[blockIdx.x];
  const int tid = threadIdx.x, lane = tid & 63;
  const int x0 = (tile % tiles_x) * kTile, y0 = (tile / tiles_x) * kTile;
  // each wave a quadrant of 8 x 8 pixels
  const int w = (int)__builtin_amdgcn_readfirstlane((uint32_t)tid >> 6);
  const int qx = (w & 1) * 8 + (lane & 7), qy = (w >> 1) * 8 + (lane >> 3);
  const int px = x0 + qx, py = y0 + qy;
  // pixel centres relative to the tile's corner
  const float fx = (float)qx + 0.5f, fy = (float)qy + 0.5f;
  const bool inside = px < W && py < H;
  float T = 1.0f, C0 = 0.0f, C1 = 0.0f, C2 = 0.0f;
  int last = 0, nbl = 0;
  bool done = !inside;
  float Tw = inside ? 1.0f : 0.0f;   // PRED: T while the pixel is blending, then 0
  const uint2 rg = ranges[tile];
  const int n = (int)(rg.y - rg.x);
  int last_start = -1;   // start of the last batch walked
  uint32_t n_bl = 0;     // blended entries listed so far
  if (tid == 0) {
    s_a[kBatch] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    s_b[kBatch] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    s_c[kBatch] = make_float4(INFINITY, 0.0f, 0.0f, 0.0f);
  }
  for (int start = 0; start < n; start += kBatch) {
    if (__syncthreads_and(done)) break;
    // the previous batch's blended entries join the list, this batch's flags start at zero
    if (blended && start > 0)
      append_blended<NT>(s_taken, s_id, s_wcnt, start - kBatch, n, blended + rg.x, n_bl, tid);
    s_taken[tid] = 0;
    bool finite = true;   // PRED: every staged colour is
    uint32_t reach = 0u;
    if (start + tid < n) {
      const uint32_t g = values[rg.x + start + tid];
      s_id[tid] = g;
      float4 a, b, c;
      stage_entry(xyab, cop, blue, g, x0, y0, a, b, c);
      s_a[tid] = a;
      s_b[tid] = b;
      s_c[tid] = c;
      reach = reach_mask(a, b, c.x);
      finite = isfinite(b.z) && isfinite(b.w) && isfinite(c.y);
    }
    s_reach[tid] = (uint8_t)reach;
    if (PRED)
      finite = __syncthreads_and(finite);
    else
      __syncthreads();
    // this wave's entries, in list order and filled up to whole groups
    int cnt = 0;
#pragma unroll
    for (int k = 0; k < kBatch; k += 64) {
      const bool in = (s_reach[k + lane] >> w) & 1u;
      const unsigned long long m = __ballot(in);
      if (in)
        s_off[w][cnt + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] =
            (uint16_t)((k + lane) * sizeof(float4));
      cnt += (int)__popcll(m);
    }
    if (lane < kFill) s_off[w][cnt + lane] = (uint16_t)(kBatch * sizeof(float4));
    wave_lds_fence();
    int last_at = -1;   // the last entry taken in this batch, as a place in the wave's list
    // the offsets of the group at place j0 of the wave's list, two entries a word
    const auto offsets = [&](int j0, uint32_t(&off)[U / 2]) {
#pragma unroll
      for (int k = 0; k < U / 2; k += 2) {
        const uint2 o = *reinterpret_cast<const uint2 *>(&s_off[w][j0 + 2 * k]);
        off[k] = o.x;
        off[k + 1] = o.y;
      }
    };
    if constexpr (PRED) {
      struct Group {
        float al[U], c0[U], c1[U], c2[U];   // alpha (0 where the entry does not reach the pixel), colour
      };
      const auto read = [&](int j0, Group &g) {
        uint32_t off[U / 2];
        offsets(j0, off);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const uint32_t e = (u & 1 ? off[u >> 1] >> 16 : off[u >> 1] & 0xFFFFu);
          const float4 A = *reinterpret_cast<const float4 *>(reinterpret_cast<const char *>(s_a) + e);
          const float4 B = *reinterpret_cast<const float4 *>(reinterpret_cast<const char *>(s_b) + e);
          // threshold on l, blue
          const float2 BL = *reinterpret_cast<const float2 *>(reinterpret_cast<const char *>(s_c) + e);
          const float dx = fx - A.x;
          const float t = conic_column(A.w, dx, B.y);
          const float l = conic_kq(B.x, A.z, dx, fy - A.y, t);   // k q + log2 o
          const float a = fminf(kAlphaMax, alpha_from_log2(l));
          g.al[u] = l < BL.x ? 0.0f : a;
          g.c0[u] = B.z;
          g.c1[u] = B.w;
          g.c2[u] = BL.y;
        }
      };
      const auto take = [&](int j0, const Group &g) {
        uint32_t bits = 0u;   // the pixel's taken entries, the last one in bit 0
        auto walk = [&](auto finite) {
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const float Tn = fmaf(-g.al[u], Tw, Tw);
            const bool stop = Tn < kTMin;                // also once Tw is 0
            const float wgt = stop ? 0.0f : g.al[u] * Tw;
            const bool take = wgt > 0.0f;
            Tw = stop ? 0.0f : Tn;
            T = stop ? T : Tn;
            if (decltype(finite)::value) {
              C0 = fmaf(wgt, g.c0[u], C0);
              C1 = fmaf(wgt, g.c1[u], C1);
              C2 = fmaf(wgt, g.c2[u], C2);
            } else {
              C0 = take ? fmaf(wgt, g.c0[u], C0) : C0;
              C1 = take ? fmaf(wgt, g.c1[u], C1) : C1;
              C2 = take ? fmaf(wgt, g.c2[u], C2) : C2;
            }
            bits = bits + bits + (take ? 1u : 0u);
          }
        };
        if (finite)
          walk(std::true_type{});
        else
          walk(std::false_type{});
        if (bits) last_at = j0 + U - __ffs((int)bits);
        if (COUNT) nbl += __popc(bits);
        if (blended) {
          const uint32_t any = wave_or(bits);
          if (lane < U && ((any >> (U - 1 - lane)) & 1u)) s_taken[s_off[w][j0 + lane] / sizeof(float4)] = 1;
        }
        done = Tw == 0.0f;
      };
      Group g0, g1;
      if (AHEAD) read(0, g0);
      for (int j0 = 0; j0 < cnt; j0 += AHEAD ? 2 * U : U) {
        if (!__any(Tw != 0.0f)) break;
        if (AHEAD) {
          // each group is read before the one in front of it is taken: j0 < cnt here and j0 + U < cnt
          // below, so what is read lies before place cnt + 2 U, the end of the fill
          read(j0 + U, g1);
          take(j0, g0);
          if (j0 + U >= cnt || !__any(Tw != 0.0f)) break;
          read(j0 + 2 * U, g0);
          take(j0 + U, g1);
        } else {
          read(j0, g0);
          take(j0, g0);
        }
      }
    } else {
      for (int j0 = 0; j0 < cnt; j0 += U) {
        if (!__any(!done)) break;
        float l[U], thr[U], c0[U], c1[U], c2[U];
        uint32_t off[U / 2];
        offsets(j0, off);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const uint32_t e = (u & 1 ? off[u >> 1] >> 16 : off[u >> 1] & 0xFFFFu);
          const float4 A = *reinterpret_cast<const float4 *>(reinterpret_cast<const char *>(s_a) + e);
          const float4 B = *reinterpret_cast<const float4 *>(reinterpret_cast<const char *>(s_b) + e);
          // threshold on l, blue
          const float2 BL = *reinterpret_cast<const float2 *>(reinterpret_cast<const char *>(s_c) + e);
          const float dx = fx - A.x;
          const float t = conic_column(A.w, dx, B.y);
          l[u] = conic_kq(B.x, A.z, dx, fy - A.y, t);   // k q + log2 o
          thr[u] = BL.x;
          c0[u] = B.z;
          c1[u] = B.w;
          c2[u] = BL.y;
        }
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
          last_at = j0 + u;
          if (COUNT) ++nbl;
          s_taken[(u & 1 ? off[u >> 1] >> 16 : off[u >> 1] & 0xFFFFu) / sizeof(float4)] = 1;
        }
      }
    }
    if (last_at >= 0) last = start + (int)(s_off[w][last_at] / sizeof(float4)) + 1;
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

// The way by the frame's tiles and by whether the blended entries are listed; us per kernel, the table's eight
// predicated entries ahead | not ahead | four predicated | four by branches:
//                                        listed                     not listed
//   1M at 800x600, 1,900 tiles        80.0  81.9  94.2  94.8     70.7  73.4  81.0  92.7
//   1M at 1000x700, 2,772             90.0  81.1  89.7  87.0     80.7  73.5  77.0  85.4
//   500k, floor 0.0125, 1280x720     80.1  70.1  78.6  76.4     73.2  64.5  66.7  75.8
//   100k uniform, 1600x900, 5,700     81.0  65.6  68.1  67.5     74.1  60.0  60.6  67.6
//   1M at 1600x900                   125.9  98.5 105.4 100.0    115.6  90.3  92.1  98.2
//   1M at 1920x1080, 8,160           160.8 121.9 125.2 120.1    148.6 114.6 111.0 118.2
//   1M, thrice as large, 1920x1080   170.7 130.1 136.8 133.0    154.6 119.6 119.9 127.5
//   1M at 3840x2160, 32,400              -     - 376.1 356.4        -     - 330.4 350.2
//   1M, a third as large, 3840x2160      -     - 378.8 360.3        -     - 338.2 348.6
//   200k, floor 0.05, 3840x2160          -     - 367.4 361.7        -     - 328.9 351.5
// Above kFewTiles the sizes of the footprints (2 to 2,000 tiles each on average) did not matter to it.
constexpr int kFewTiles = 6144, kFewestTiles = 2048;

hipError_t launch_blend(const uint2 *ranges, const uint32_t *values, const float4 *xyab, const float4 *cop,
                        const float2 *blue, const DevCamera &cam, const float bg[3], float *image, float *final_T,
                        int32_t *n_contrib, int32_t *n_blended, uint2 *blended, uint32_t *tile_blended,
                        const uint32_t *order, hipStream_t s) {
  const int n_tiles = cam.tiles_x * cam.tiles_y;
  // eight predicated entries per group while the frame has few waves for the device, read ahead where
  // it has fewer still; beyond, four, by branches where the blended entries are listed (see the table)
  const int way = n_tiles <= kFewestTiles ? 0 : n_tiles <= kFewTiles ? 1 : blended ? 3 : 2;
  auto kernel = way == 0 ? n_blended ? k_blend<8, true, true, true> : k_blend<8, true, true, false>
                : way == 1 ? n_blended ? k_blend<8, true, false, true> : k_blend<8, true, false, false>
                : way == 2 ? n_blended ? k_blend<4, true, false, true> : k_blend<4, true, false, false>
                           : n_blended ? k_blend<4, false, false, true> : k_blend<4, false, false, false>;
  hipLaunchKernelGGL(kernel, dim3(n_tiles), dim3(kTile * kTile), 0, s, ranges, values, xyab, cop, blue, cam.W, cam.H,
                     cam.tiles_x, bg[0], bg[1], bg[2], image, final_T, n_contrib, n_blended, blended, tile_blended,
                     order);
  return hipGetLastError();
}

}  // namespace flod
