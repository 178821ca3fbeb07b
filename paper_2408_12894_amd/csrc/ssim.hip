// Training loss: L1 plus SSIM (section Implementation: the backbone's L1 and SSIM losses).
//
//   F(z)     11 x 11 Gaussian window (sigma 1.5, normalised, separable), zeros outside the image
//   moments  mu_x = F(x), mu_y = F(y), E_xx = F(xx), E_yy = F(yy), E_xy = F(xy)
//   S        (2 mu_x mu_y + C1)(2 s_xy + C2) / ((mu_x^2 + mu_y^2 + C1)(s_xx + s_yy + C2)),
//            s_xx = E_xx - mu_x^2, s_yy = E_yy - mu_y^2, s_xy = E_xy - mu_x mu_y
//   loss     (1 - lam) mean|x - y| + lam (1 - mean S)
//
// Only the sum s_xx + s_yy enters S, so four windowed sums suffice: x, y, xx + yy and xy.
//
// Forward: one workgroup per 240 x 16 pixels and channel, in four steps of four rows. Vertical
// pass: thread t holds 14 rows of column t of the tile and its halo (consecutive threads read
// consecutive addresses; each step reads four new rows, while the step before is in its
// horizontal pass) and writes the four windowed column sums (FP64) of four rows to LDS.
// Horizontal pass: each thread takes four consecutive pixels of a row, so that an LDS value read
// once serves up to four sums. Each pixel then writes the partial
// derivatives of S with respect to mu_x, E_xx and E_xy (FP32, 12 B per channel-pixel), and the
// workgroup writes its sums of S and |x - y| (FP64) for a fixed-order final reduction.
// Backward: the same tiling filters the three derivative maps (the window is symmetric, so F
// is its own adjoint) and combines them: dL/dx = c (F(d_mu) + 2 x F(d_xx) + y F(d_xy)) plus
// the L1 term (1 - lam) sign(x - y) / n, c = -lam / n, times the incoming loss gradient.
// All sums are FP64; inputs and outputs FP32.
//
// Bound: FP64 issue (about 170 instructions per channel-pixel forward, 110 backward), then HBM.
// With 16 x 16 tiles, a 26 x 26 halo, five sums and one output per thread in both passes (11
// LDS reads of each map per output) the kernels took 175 + 114 us at 3 x 1920 x 1080, and the
// reduction of the 24,480 workgroup sums 26 us; now 57 + 44 + 5 us.
#include "flod_internal.h"

namespace flod {

constexpr int kSsimR = 5;                            // window radius
// Outputs per thread in either pass. Eight need a third less LDS and conversion work per pixel
// but 66 KB of LDS and 176 registers: two waves per SIMD, 107 us forward at 3 x 1920 x 1080.
constexpr int kSsimRun = 4;
constexpr int kSsimOut = kBlock - 16;                // pixels per row of a tile (their halo fits kBlock)
constexpr int kSsimSteps = 4;                        // most steps of kSsimRun rows per workgroup
constexpr int kSsimSpan = kSsimRun + 2 * kSsimR;     // inputs of kSsimRun outputs
// a row's pitch of 1 modulo 16 doubles: the 64 lanes of a horizontal read (four rows, 16 runs of
// four) spread evenly over the banks
constexpr int kSsimPitch = kBlock + 1;
constexpr int kLossTile = 16;                        // tile edge the loss's size limit counts in
constexpr double kC1 = 0.01 * 0.01;
constexpr double kC2 = 0.03 * 0.03;

struct SsimArgs {
  const float *x, *y;
  int C, H, W, tiles_x, steps;
  double lam, inv_n;
  double g[2 * kSsimR + 1];
};

// One input of a run's windowed sums: input i adds to the outputs within the window's radius.
template <int MAPS>
__device__ __forceinline__ void window_add(double (&acc)[MAPS][kSsimRun], const double (&v)[MAPS], int i,
                                           const double (&g)[2 * kSsimR + 1]) {
#pragma unroll
  for (int o = 0; o < kSsimRun; ++o) {
    const int k = i - o;
    if (k < 0 || k > 2 * kSsimR) continue;
#pragma unroll
    for (int m = 0; m < MAPS; ++m) acc[m][o] = fma(g[k], v[m], acc[m][o]);
  }
}

template <int MAPS>
using SsimColumns = double[MAPS][kSsimRun][kSsimPitch];

// The horizontal pass of one thread: its run of a row from the column sums.
template <int MAPS>
__device__ __forceinline__ void window_rows(const SsimColumns<MAPS> &s, int row, int run,
                                            const double (&g)[2 * kSsimR + 1], double (&acc)[MAPS][kSsimRun]) {
#pragma unroll
  for (int m = 0; m < MAPS; ++m)
#pragma unroll
    for (int o = 0; o < kSsimRun; ++o) acc[m][o] = 0.0;
#pragma unroll
  for (int i = 0; i < kSsimSpan; ++i) {
    double v[MAPS];
#pragma unroll
    for (int m = 0; m < MAPS; ++m) v[m] = s[m][row][run * kSsimRun + i];
    window_add<MAPS>(acc, v, i, g);
  }
}

// Rows gy .. gy + N - 1 of column gx of a plane, the nearest inside it for those outside;
// inside_rows makes those zero. Two steps, since a load whose value is only selected under a
// condition becomes a branch around it and its own wait: the values pass through an empty asm
// where they are first used, which keeps the loads together and waits there only, and are then
// masked bit by bit.
template <int N>
__device__ __forceinline__ void load_column(const float *__restrict__ src, int W, int H, int gx, int gy, float (&v)[N]) {
  // a 32-bit byte offset from the row, whose address is the same in every thread (and in scalar
  // registers: the tile's place comes from the block's, not from a division)
  const uint32_t at = 4u * (uint32_t)min(max(gx, 0), W - 1);
#pragma unroll
  for (int i = 0; i < N; ++i)
    v[i] = *reinterpret_cast<const float *>(
        reinterpret_cast<const char *>(src + (int64_t)min(max(gy + i, 0), H - 1) * W) + at);
}

template <int N>
__device__ __forceinline__ void inside_rows(float (&v)[N], int W, int H, int gx, int gy) {
  uint32_t in = gx >= 0 && gx < W ? ~0u : 0u;
  asm volatile("" : "+v"(in));
#pragma unroll
  for (int i = 0; i < N; ++i) asm volatile("" : "+v"(v[i]));
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const uint32_t row = gy + i >= 0 && gy + i < H ? ~0u : 0u;   // the same in every thread
    v[i] = __uint_as_float(__float_as_uint(v[i]) & (in & row));
  }
}

// The held rows moved up by one step, the new ones behind them.
__device__ __forceinline__ void next_rows(float (&v)[kSsimSpan], const float (&add)[kSsimRun]) {
#pragma unroll
  for (int i = 0; i < kSsimSpan; ++i) v[i] = i + kSsimRun < kSsimSpan ? v[i + kSsimRun] : add[i + kSsimRun - kSsimSpan];
}

// Four consecutive values of a row, those inside it: one 16-byte store when whole and aligned.
__device__ __forceinline__ void store_run(float *__restrict__ dst, const float (&v)[kSsimRun], int n, bool vec) {
  static_assert(kSsimRun == 4, "a run is one float4");
  if (vec && n >= kSsimRun) {
    *reinterpret_cast<float4 *>(dst) = make_float4(v[0], v[1], v[2], v[3]);
  } else {
#pragma unroll
    for (int o = 0; o < kSsimRun; ++o)
      if (o < n) dst[o] = v[o];
  }
}

template <bool WITH_GRAD>
__global__ __launch_bounds__(kBlock) void k_ssim_fwd(SsimArgs a, float *gmap, bool vec, double2 *partials) {
  __shared__ SsimColumns<4> s_col;
  __shared__ double red[2][kBlock / 64];
  const int ch = blockIdx.z, tid = threadIdx.x;
  const int x0 = blockIdx.x * kSsimOut, yt = blockIdx.y * kSsimRun * a.steps;
  const int64_t plane = (int64_t)a.H * a.W, stride = (int64_t)a.C * plane;
  const float *__restrict__ xs = a.x + ch * plane, *__restrict__ ys = a.y + ch * plane;
  const int row = tid % kSsimRun, run = tid / kSsimRun;
  double s_sum = 0.0, l1_sum = 0.0;
  const int gx = x0 - kSsimR + tid;
  float xv[kSsimSpan], yv[kSsimSpan], xn[kSsimRun], yn[kSsimRun];
  load_column(xs, a.W, a.H, gx, yt - kSsimR, xv);
  load_column(ys, a.W, a.H, gx, yt - kSsimR, yv);
  inside_rows(xv, a.W, a.H, gx, yt - kSsimR);
  inside_rows(yv, a.W, a.H, gx, yt - kSsimR);
  for (int step = 0; step < a.steps; ++step) {
    const int y0 = yt + step * kSsimRun;
    if (y0 >= a.H) break;   // the same in every thread
    const int new_y = y0 + kSsimRun + kSsimR;   // the next step's new rows
    load_column(xs, a.W, a.H, gx, new_y, xn);
    load_column(ys, a.W, a.H, gx, new_y, yn);
    {
      double acc[4][kSsimRun];
#pragma unroll
      for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int o = 0; o < kSsimRun; ++o) acc[m][o] = 0.0;
      double l1 = 0.0;
#pragma unroll
      for (int i = 0; i < kSsimSpan; ++i) {
        const double x = xv[i], y = yv[i];
        const double v[4] = {x, y, fma(x, x, y * y), x * y};
        window_add<4>(acc, v, i, a.g);
        if (i >= kSsimR && i < kSsimR + kSsimRun) l1 += fabs(x - y);   // zero outside the image
      }
      if (tid >= kSsimR && tid < kSsimR + kSsimOut) l1_sum += l1;
#pragma unroll
      for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int o = 0; o < kSsimRun; ++o) s_col[m][o][tid] = acc[m][o];
    }
    lds_barrier();
    const int px = x0 + run * kSsimRun, py = y0 + row;
    const int n = min(kSsimRun, a.W - px);
    if (run < kSsimOut / kSsimRun && py < a.H && n > 0) {
      double f[4][kSsimRun];
      window_rows<4>(s_col, row, run, a.g, f);
      float d_mu[kSsimRun], d_xx[kSsimRun], d_xy[kSsimRun];
#pragma unroll
      for (int o = 0; o < kSsimRun; ++o) {
        const double mx = f[0][o], my = f[1][o];
        // equal images give A = Cc and B = D exactly, and S = 1: m2 = 2 mxy, f2 = 2 f3, and
        // the quotient's correction below rounds to 1
        const double m2 = mx * mx + my * my, mxy = mx * my;
        const double A = fma(2.0, mxy, kC1), B = fma(2.0, f[3][o] - mxy, kC2);
        const double Cc = m2 + kC1, D = (f[2][o] - m2) + kC2;
        const double CD = Cc * D, AB = A * B, r = 1.0 / CD;
        const double S0 = AB * r, S = fma(fma(-S0, CD, AB), r, S0);   // AB / CD
        const double Ar = A * r;
        if (o < n) s_sum += S;
        if (WITH_GRAD) {
          // 1 / D = Cc r, 1 / Cc = D r
          const double sxD = S * (Cc * r), Br = B * r;
          d_xx[o] = (float)(-sxD);
          d_xy[o] = (float)(2.0 * Ar);
          d_mu[o] = (float)(2.0 * (my * (Br - Ar) + mx * (sxD - S * (D * r))));
        }
      }
      if (WITH_GRAD) {
        float *dst = gmap + ch * plane + (int64_t)py * a.W + px;
        store_run(dst, d_mu, n, vec);
        store_run(dst + stride, d_xx, n, vec);
        store_run(dst + 2 * stride, d_xy, n, vec);
      }
    }
    lds_barrier();
    inside_rows(xn, a.W, a.H, gx, new_y);
    inside_rows(yn, a.W, a.H, gx, new_y);
    next_rows(xv, xn);
    next_rows(yv, yn);
  }
  for (int off = 32; off > 0; off >>= 1) {
    s_sum += __shfl_down(s_sum, off, 64);
    l1_sum += __shfl_down(l1_sum, off, 64);
  }
  if ((tid & 63) == 0) {
    red[0][tid >> 6] = s_sum;
    red[1][tid >> 6] = l1_sum;
  }
  __syncthreads();
  if (tid == 0) {
    double s = 0, l = 0;
    for (int w = 0; w < kBlock / 64; ++w) {
      s += red[0][w];
      l += red[1][w];
    }
    partials[((int64_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x] = make_double2(s, l);
  }
}

// Fixed-order reduction of the workgroup sums (one workgroup): deterministic loss. Four sums per
// thread are loaded together.
constexpr int kReduceThreads = 1024;

__global__ __launch_bounds__(kReduceThreads) void k_ssim_reduce(const double2 *__restrict__ partials, int64_t count,
                                                                double lam, double inv_n, double *loss) {
  __shared__ double red[2][kReduceThreads / 64];
  double s = 0, l = 0;
  for (int64_t i = threadIdx.x; i < count; i += 4 * kReduceThreads) {
    double2 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      v[u] = i + u * kReduceThreads < count ? partials[i + u * kReduceThreads] : make_double2(0.0, 0.0);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      s += v[u].x;
      l += v[u].y;
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
    s += __shfl_down(s, off, 64);
    l += __shfl_down(l, off, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = s;
    red[1][threadIdx.x >> 6] = l;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double st = 0, lt = 0;
    for (int w = 0; w < kReduceThreads / 64; ++w) {
      st += red[0][w];
      lt += red[1][w];
    }
    loss[0] = (1.0 - lam) * (lt * inv_n) + lam * (1.0 - st * inv_n);
  }
}

// Three waves per SIMD: unbounded it took 182 registers (48 us against 44 at 3 x 1920 x 1080; at
// four 89 us, with spills all over; at three an address spills, loaded back once a step).
__global__ __launch_bounds__(kBlock, 3) void k_ssim_bwd(SsimArgs a, const float *__restrict__ gmap, bool vec,
                                                     const double *dloss, float *__restrict__ dx) {
  __shared__ SsimColumns<3> s_col;
  const int ch = blockIdx.z, tid = threadIdx.x;
  const int x0 = blockIdx.x * kSsimOut, yt = blockIdx.y * kSsimRun * a.steps;
  const int64_t plane = (int64_t)a.H * a.W, stride = (int64_t)a.C * plane;
  const float *__restrict__ gm = gmap + ch * plane;
  const int row = tid % kSsimRun, run = tid / kSsimRun;
  const double up = dloss ? dloss[0] : 1.0;
  const double c = -a.lam * a.inv_n * up, c1 = (1.0 - a.lam) * a.inv_n * up;
  const int gx = x0 - kSsimR + tid;
  float v0[kSsimSpan], v1[kSsimSpan], v2[kSsimSpan], n0[kSsimRun], n1[kSsimRun], n2[kSsimRun];
  load_column(gm, a.W, a.H, gx, yt - kSsimR, v0);
  load_column(gm + stride, a.W, a.H, gx, yt - kSsimR, v1);
  load_column(gm + 2 * stride, a.W, a.H, gx, yt - kSsimR, v2);
  inside_rows(v0, a.W, a.H, gx, yt - kSsimR);
  inside_rows(v1, a.W, a.H, gx, yt - kSsimR);
  inside_rows(v2, a.W, a.H, gx, yt - kSsimR);
  for (int step = 0; step < a.steps; ++step) {
    const int y0 = yt + step * kSsimRun;
    if (y0 >= a.H) break;   // the same in every thread
    const int new_y = y0 + kSsimRun + kSsimR;   // the next step's new rows
    load_column(gm, a.W, a.H, gx, new_y, n0);
    load_column(gm + stride, a.W, a.H, gx, new_y, n1);
    load_column(gm + 2 * stride, a.W, a.H, gx, new_y, n2);
    const int px = x0 + run * kSsimRun, py = y0 + row;
    const int n = min(kSsimRun, a.W - px);
    const bool mine = run < kSsimOut / kSsimRun && py < a.H && n > 0;
    const int64_t at = ch * plane + (int64_t)py * a.W + px;
    float xv[kSsimRun], yv[kSsimRun];   // this thread's pixels, loaded ahead of the barrier
    if (mine) {
      if (vec && n >= kSsimRun) {
        const float4 x4 = *reinterpret_cast<const float4 *>(a.x + at), y4 = *reinterpret_cast<const float4 *>(a.y + at);
        xv[0] = x4.x; xv[1] = x4.y; xv[2] = x4.z; xv[3] = x4.w;
        yv[0] = y4.x; yv[1] = y4.y; yv[2] = y4.z; yv[3] = y4.w;
      } else {
#pragma unroll
        for (int o = 0; o < kSsimRun; ++o) {
          xv[o] = a.x[at + min(o, n - 1)];
          yv[o] = a.y[at + min(o, n - 1)];
        }
      }
    }
    // one map after the other: interleaved, the three hold twice the registers
    auto columns = [&](const float (&v)[kSsimSpan], int m) {
      double acc[1][kSsimRun] = {};
#pragma unroll
      for (int i = 0; i < kSsimSpan; ++i) {
        const double in[1] = {(double)v[i]};
        window_add<1>(acc, in, i, a.g);
      }
#pragma unroll
      for (int o = 0; o < kSsimRun; ++o) s_col[m][o][tid] = acc[0][o];
      __builtin_amdgcn_sched_barrier(0);
    };
    columns(v0, 0);
    columns(v1, 1);
    columns(v2, 2);
    lds_barrier();
    if (mine) {
      double f[3][kSsimRun];
      window_rows<3>(s_col, row, run, a.g, f);
      float d[kSsimRun];
#pragma unroll
      for (int o = 0; o < kSsimRun; ++o) {
        const double x = xv[o], y = yv[o];
        const double l1 = x > y ? c1 : x < y ? -c1 : 0.0;
        d[o] = (float)fma(c, fma(2.0 * x, f[1][o], fma(y, f[2][o], f[0][o])), l1);
      }
      store_run(dx + at, d, n, vec);
    }
    lds_barrier();
    inside_rows(n0, a.W, a.H, gx, new_y);
    inside_rows(n1, a.W, a.H, gx, new_y);
    inside_rows(n2, a.W, a.H, gx, new_y);
    next_rows(v0, n0);
    next_rows(v1, n1);
    next_rows(v2, n2);
  }
}

static SsimArgs ssim_args(const float *x, const float *y, int C, int H, int W, float lam) {
  SsimArgs a;
  a.x = x;
  a.y = y;
  a.C = C;
  a.H = H;
  a.W = W;
  a.tiles_x = (W + kSsimOut - 1) / kSsimOut;
  a.lam = (double)lam;
  a.inv_n = 1.0 / ((double)C * (double)H * (double)W);
  double sum = 0.0;
  for (int k = 0; k <= 2 * kSsimR; ++k) {
    const double d = (double)(k - kSsimR);
    a.g[k] = std::exp(-(d * d) / (2.0 * 1.5 * 1.5));
    sum += a.g[k];
  }
  for (int k = 0; k <= 2 * kSsimR; ++k) a.g[k] /= sum;
  return a;
}

constexpr int64_t kSsimFew = 1024;

int64_t ssim_blocks(int C, int H, int W) {
  return std::max<int64_t>(kSsimFew, (int64_t)((W + kLossTile - 1) / kLossTile) * ((H + kLossTile - 1) / kLossTile) * C);
}

// Steps per workgroup: four, which read 26 rows for 16, or fewer (14 rows for four) for images
// that would leave the device mostly idle with them (up to kSsimFew workgroups; as few as an image's
// 16 x 16 tiles, 1 x 16 x 16 took 22.8 us forward and backward, one workgroup's four steps, and 3 x 500 x 16
// 24.8, now 16.4 and 15.6). There are never more workgroups than ssim_blocks (the caller's room for their
// sums). Narrow high images keep most of a tile's columns idle (3 x 8000 x 16 62 us, of 16 x 16 tiles 27): going
// through them down their columns took 35, and leaving idle waves out spilled in the backward (44 -> 53 us at
// 3 x 1920 x 1080).
static dim3 ssim_grid(SsimArgs &a) {
  auto count = [&](int steps) {
    return (int64_t)a.tiles_x * ((a.H + kSsimRun * steps - 1) / (kSsimRun * steps)) * a.C;
  };
  static_assert(kSsimRun * kSsimSteps >= kLossTile && kSsimOut >= kLossTile, "ssim_blocks bounds the workgroups");
  a.steps = kSsimSteps;
  while (a.steps > 1 && count(a.steps / 2) <= kSsimFew) a.steps /= 2;
  return dim3((unsigned)a.tiles_x, (unsigned)(count(a.steps) / a.C / a.tiles_x), (unsigned)a.C);
}

// 16-byte stores: every row of every plane has to start 16-byte aligned
static bool vec_rows(const void *p, int W) { return W % 4 == 0 && reinterpret_cast<uintptr_t>(p) % 16 == 0; }

hipError_t launch_ssim_forward(const float *x, const float *y, int C, int H, int W, float lam, double *loss,
                               float *gmap, double2 *partials, hipStream_t s) {
  SsimArgs a = ssim_args(x, y, C, H, W, lam);
  const dim3 grid = ssim_grid(a);
  if (gmap)
    hipLaunchKernelGGL(k_ssim_fwd<true>, grid, dim3(kBlock), 0, s, a, gmap, vec_rows(gmap, W), partials);
  else
    hipLaunchKernelGGL(k_ssim_fwd<false>, grid, dim3(kBlock), 0, s, a, gmap, false, partials);
  hipLaunchKernelGGL(k_ssim_reduce, dim3(1), dim3(kReduceThreads), 0, s, partials, (int64_t)grid.x * grid.y * grid.z, a.lam,
                     a.inv_n, loss);
  return hipGetLastError();
}

hipError_t launch_ssim_backward(const float *x, const float *y, int C, int H, int W, float lam, const float *gmap,
                                const double *dloss, float *dx, hipStream_t s) {
  SsimArgs a = ssim_args(x, y, C, H, W, lam);
  const dim3 grid = ssim_grid(a);
  hipLaunchKernelGGL(k_ssim_bwd, grid, dim3(kBlock), 0, s, a, gmap,
                     vec_rows(dx, W) && vec_rows(x, W) && vec_rows(y, W), dloss, dx);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Plain L1 loss, mean|x - y| over `count` elements (the image loss of the training step):
// a grid-stride FP64 sum per workgroup, then the fixed-order reduction above; the backward
// writes sign(x - y) / count times the incoming loss gradient.
// ---------------------------------------------------------------------------------------
constexpr int kL1Blocks = 1024;

__global__ __launch_bounds__(kBlock) void k_l1_fwd(const float4 *__restrict__ x, const float4 *__restrict__ y,
                                                   const float *__restrict__ xs, const float *__restrict__ ys,
                                                   int64_t n4, int64_t n, double2 *partials) {
  __shared__ double red[kBlock / 64];
  double acc = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n4; i += (int64_t)gridDim.x * kBlock) {
    const float4 a = x[i], b = y[i];
    acc += (double)fabsf(a.x - b.x) + (double)fabsf(a.y - b.y) + (double)fabsf(a.z - b.z) +
           (double)fabsf(a.w - b.w);
  }
  if (blockIdx.x == 0)
    for (int64_t i = n4 * 4 + threadIdx.x; i < n; i += kBlock) acc += (double)fabsf(xs[i] - ys[i]);
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int w = 0; w < kBlock / 64; ++w) t += red[w];
    partials[blockIdx.x] = make_double2(0.0, t);
  }
}

__global__ __launch_bounds__(kBlock) void k_l1_bwd(const float *__restrict__ x, const float *__restrict__ y,
                                                   int64_t n, double inv_n, const double *dloss,
                                                   float *__restrict__ dx) {
  const float scale = (float)(dloss ? inv_n * dloss[0] : inv_n);
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock) {
    const float t = x[i] - y[i];
    dx[i] = t > 0.0f ? scale : (t < 0.0f ? -scale : 0.0f);
  }
}

int64_t l1_blocks() { return kL1Blocks; }

hipError_t launch_l1_forward(const float *x, const float *y, int64_t n, double *loss, double2 *partials,
                             hipStream_t s) {
  const bool vec = (reinterpret_cast<uintptr_t>(x) % 16 == 0) && (reinterpret_cast<uintptr_t>(y) % 16 == 0);
  const int64_t n4 = vec ? n / 4 : 0;
  hipLaunchKernelGGL(k_l1_fwd, dim3(kL1Blocks), dim3(kBlock), 0, s, reinterpret_cast<const float4 *>(x),
                     reinterpret_cast<const float4 *>(y), x, y, n4, n, partials);
  // (1 - lam) L1 + lam (1 - S) with lam = 0 and the S sums zero: the mean of |x - y|
  hipLaunchKernelGGL(k_ssim_reduce, dim3(1), dim3(kReduceThreads), 0, s, partials, (int64_t)kL1Blocks, 0.0,
                     1.0 / (double)n, loss);
  return hipGetLastError();
}

hipError_t launch_l1_backward(const float *x, const float *y, int64_t n, const double *dloss, float *dx,
                              hipStream_t s) {
  const int64_t blocks = std::min<int64_t>((n + kBlock - 1) / kBlock, 4096);
  hipLaunchKernelGGL(k_l1_bwd, dim3((unsigned)blocks), dim3(kBlock), 0, s, x, y, n, 1.0 / (double)n, dloss, dx);
  return hipGetLastError();
}

}  // namespace flod
