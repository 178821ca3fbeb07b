// Internal declarations shared by the kernels and the host orchestration of libflod.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/flod.h"

namespace flod {

constexpr int kTile = FLOD_TILE;          // 16x16 pixel tiles
constexpr int kMaxSide = 16384;           // largest frame side
constexpr int kBlock = 256;               // threads per workgroup (4 wave64)
constexpr int kRadixBits = 8;
constexpr int kRadix = 1 << kRadixBits;   // 256 buckets per radix pass
// The depth sort's digits: the bits of a rendered depth are at least kDepthBase (0.125; the near plane
// is 0.2), and below 8192 they exceed it by less than 2^27: three passes of 9 bits. A frame with
// a depth beyond takes four passes of 8 (kDepthFarBits). Three against four passes: 65 against
// 78 us at 857k keys, 26 against 35 at 8k.
constexpr int kDepthBits = 9, kDepthRadix = 1 << kDepthBits, kDepthFarBits = 31;
constexpr uint32_t kDepthBase = 0x3E000000u;
// A frame sorted again after three passes pays for both sorts, so the next kFarHold frames start with
// four: a camera that alternates between near and far views pays once.
constexpr int kFarHold = 32;
constexpr int64_t kSmallSort = 8192;      // candidates up to which one workgroup sorts the frame
// Keys per thread in a radix pass: 2048-key workgroups below kRadixBigSort keys of capacity, 3072 up to
// kRadixHugeSort, 4096 from there on. The grids are sized for the capacity, but after the first pass only the
// visible keys are left: larger workgroups gain where most are visible and lose where few are. The
// depth sort with 8 | 12 | 16 keys per thread, us, most candidates visible, then a tenth of them: 1.5M 86 87
// 91, 52 57 63; 3M 144 134 131, 67 70 75; 4.5M 203 188 187, 80 80 87; 10M 12 against 16 368 365, 117 121; 24M 889
// 850, 221 216; selected from 2.5M (a sixth visible) 63 64 68, from 4.2M 89 83 89. Overlap pruning as a
// whole differs by less than 2% between them.
constexpr int kSortItems = 8, kSortItemsBig = 12, kSortItemsHuge = 16;
constexpr int64_t kRadixBigSort = 4 << 20, kRadixHugeSort = 32 << 20;
constexpr int kSuper = 8;                 // a supertile is kSuper x kSuper tiles (one bit each of a 64-bit mask)
constexpr int kSuperWindow = 512;         // supertiles whose pairs a workgroup places
constexpr int kPairBlock = 256;           // depth-sorted Gaussians a workgroup of the pair kernels takes at once
constexpr int kChunk = 256;               // pairs of one supertile expanded by one workgroup
constexpr int kSpanBox = 16;              // largest footprint (tiles a side) whose row spans are stored
constexpr int kPairRectMax = 16;          // largest rectangle (in supertiles) listed whole
// A Gaussian's tile rectangle as the binning reads it: x0 | y0 << 16 and x1 | y1 << 16 (frames have
// at most 1024 x 1024 tiles) with what else it has to know: the footprint is the whole rectangle;
// its supertiles are listed row by row instead of the whole rectangle's; its row spans, or of a
// banded one its supertile rows' columns, are stored (kSpanNone), counted from a column that many
// (four bits at kRectBefore of the first word) before the rectangle's first.
constexpr uint32_t kRectFull = 1u << 31, kRectBanded = 1u << 30, kRectBoxed = 1u << 29;
constexpr uint32_t kRectCorner = 0x0FFFFFFFu, kRectBefore = 10;
constexpr size_t kGaussianBytes = (3 + 3 + 4 + 1 + FLOD_SH_COEFFS * 3) * 4;   // 236 B per stored Gaussian
constexpr unsigned long long kPruneMaxScan = 1ull << 36;   // overlap-pruning neighbour-scan limit

// Rasterizer conventions (3DGS framework): near plane, EWA dilation, Jacobian clamp at 1.3x the half field of view, alpha clamp, alpha floor,
// transmittance floor, support cut q <= 9.
constexpr float kNearZ = 0.2f;
constexpr float kDilate = 0.3f;
constexpr float kFovClamp = 1.3f;
// Depth key of a candidate that is not rendered (culled or not selected): above every FP32
// depth bits of a positive depth, and skipped by the depth sort's first pass.
constexpr uint32_t kDepthNone = 0xFFFFFFFFu;
constexpr float kAlphaMax = 0.99f;
constexpr float kAlphaMin = 1.0f / 255.0f;
constexpr float kTMin = 1e-4f;
constexpr float kQCut = 9.0f;
constexpr double kNearZD = 0.2;
constexpr double kDilateD = 0.3;
constexpr double kFovClampD = 1.3;

struct DevCamera {
  float R[9], t[3], campos[3];
  float fx, fy, cx, cy;
  int W, H, tiles_x, tiles_y;
};

struct DevLevel {
  const float *means, *log_scales, *quats, *logits, *sh;
  int64_t offset, n;
  float s_min;
  float lo2, hi2;     // eq. 6 band, squared; used only when selecting
};

struct PreParams {
  DevLevel lv[FLOD_MAX_LEVELS];
  int n_levels;
  int select;
  int sh_degree;
  float logit_min;    // opacity cull: logit < logit_min  <=>  opacity < 1/255
  float centre[3];
  DevCamera cam;
  int64_t n_total;
};

// Per-candidate outputs of the preprocess (structure of arrays).
struct PreOut {
  float4 *xyab;       // mu'x, mu'y, conic a, conic b
  float4 *cop;        // conic c, opacity, red, green
  float2 *blue;       // blue, packed bf16 residuals of mu' (bits)
  uint32_t *depth;    // FP32 bits of the view-space depth
  float *qsup;        // support bound Q_g
  uint32_t *tiles;    // tiles touched, 0 when culled or not selected
  uint2 *rect;        // tile rectangle and flags of rendered candidates (kRectFull ...)
  uint4 *spans;       // row spans of those with kRectBoxed (see kSpanNone)
  uint4 *block_sums;  // per workgroup: visible candidates, tiles, (supertile, Gaussian) pairs and
                      // candidates beyond the depth sort's three passes
  unsigned long long *n_selected;   // per-level selected counts (may be null)
  float4 *shjac;      // three planes of n_total float4, per visible candidate the colour's Jacobian in
                      // the unit view direction, J[ch][a] row-major, then the three colours before the
                      // clamp (J00 J01 J02 J10 | J11 J12 J20 J21 | J22 c0 c1 c2); may be null
};

// What the binning reads of a candidate besides its rectangle.
struct BinIn {
  const float4 *xyab, *cop;
  const float *qsup;
  const uint4 *spans;
};

// One attribute array of a level in an Adam step: parameter, gradient and the two moment
// arrays (same length), its first float4 slot in the launch and its learning rate.
struct AdamSeg {
  float *p;
  const float *g;
  float *m, *v;
  int64_t len;      // floats
  int64_t first4;   // first float4 slot of the segment
  float lr;         // for the SH segment: the degree-0 rate
  int vec;          // all four arrays 16-byte aligned
};

struct AdamArgs {
  AdamSeg seg[5];   // means, log_scales, quats, opacity logits, SH
  float lr_sh_rest;
  float b1, b2, omb1, omb2;   // beta1, beta2, 1 - beta1, 1 - beta2
  float inv_bc1, inv_bc2;     // 1 / (1 - beta^t), formed in FP64 and rounded once
  float eps;
  int64_t total4;
};

// Counters in device memory (one small array per context).
enum : int {
  kCntVisible = 0,      // u32 count of visible candidates
  kCntTotal64 = 2,      // u64 count of instances (or other totals; two u32 slots: 2, 3)
  kCntPairs64 = 4,      // u64 count of (supertile, Gaussian) pairs (slots 4, 5)
  kCntPairs = 6,        // u32 count of pairs; 0 when instances or pairs exceed their buffers
  kCntChunks = 7,       // u32 count of chunks of pairs
  kCntFar = 1,          // u32 count of visible candidates beyond the depth sort's three passes
  kCntKept = 8,         // u32 counts of the Gaussians a compaction keeps, one per level (slots 8 .. 15)
  kCntSlots = 16
};

// Sums of the preprocess's per-workgroup counts, taken by one workgroup of kBlock threads:
// visible candidates, instances K and pairs P, to the device counters and, when host_out is
// given (coherent host memory), to the host. kCntPairs receives P when K <= cap_k and
// P <= cap_p and 0 otherwise: kernels sized for those capacities read it and then do nothing.
// near_only: 0 too when there are far candidates, whose order three passes leave wrong (the host sorts
// again, with four, and takes the totals without it).
// host_out receives six 64-bit words, each host_seq in its high half and in its low half the
// visible count, the low and high halves of K and of P, and the count of far ones: system-scope stores of whole words,
// so a host that polls them sees every word either old or complete and needs neither a copy
// nor an event.
struct FrameTotals {
  const uint4 *sums;
  int nb;
  uint32_t *counters;
  unsigned long long cap_k, cap_p;
  unsigned long long *host_out;
  uint32_t host_seq;
  bool near_only;
};

__device__ __forceinline__ void frame_totals(const FrameTotals &t) {
  constexpr int U = 8, W = kBlock / 64;
  __shared__ unsigned long long s_sum[4][W];
  unsigned long long v = 0, k = 0, p = 0, far = 0;
  for (int i0 = threadIdx.x; i0 < t.nb; i0 += kBlock * U) {
    uint4 x[U];   // loaded together
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * kBlock;
      x[u] = i < t.nb ? t.sums[i] : make_uint4(0u, 0u, 0u, 0u);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      v += x[u].x;
      k += x[u].y;
      p += x[u].z;
      far += x[u].w;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    v += __shfl_xor(v, o, 64);
    k += __shfl_xor(k, o, 64);
    p += __shfl_xor(p, o, 64);
    far += __shfl_xor(far, o, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    s_sum[0][threadIdx.x >> 6] = v;
    s_sum[1][threadIdx.x >> 6] = k;
    s_sum[2][threadIdx.x >> 6] = p;
    s_sum[3][threadIdx.x >> 6] = far;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  v = k = p = far = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    v += s_sum[0][w];
    k += s_sum[1][w];
    p += s_sum[2][w];
    far += s_sum[3][w];
  }
  t.counters[kCntVisible] = (uint32_t)v;
  t.counters[kCntFar] = (uint32_t)far;
  *reinterpret_cast<unsigned long long *>(t.counters + kCntTotal64) = k;
  *reinterpret_cast<unsigned long long *>(t.counters + kCntPairs64) = p;
  t.counters[kCntPairs] = k <= t.cap_k && p <= t.cap_p && !(t.near_only && far) ? (uint32_t)p : 0u;
  if (t.host_out) {
    const unsigned long long tag = (unsigned long long)t.host_seq << 32;
    const unsigned long long w[6] = {tag | v, tag | (k & 0xFFFFFFFFull), tag | (k >> 32), tag | (p & 0xFFFFFFFFull),
                                     tag | (p >> 32), tag | far};
#pragma unroll
    for (int i = 0; i < 6; ++i) __hip_atomic_store(&t.host_out[i], w[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// Block of a workgroup: workgroups go to the 8 XCDs round-robin, and each XCD takes runs of
// kXcdRun consecutive blocks. What adjacent blocks write then shares cache lines inside one
// XCD's L2 and moves as whole lines (spread over the 8 XCDs, the radix histograms went out as 8
// partial writes of every line: 8x their bytes).
constexpr uint32_t kXcdRun = 16;

__device__ __forceinline__ uint32_t xcd_block(uint32_t wg) {
  const uint32_t x = wg % 8u, j = wg / 8u;
  return (j / kXcdRun) * (8u * kXcdRun) + x * kXcdRun + (j % kXcdRun);
}

inline unsigned xcd_grid(int64_t blocks) {
  const int64_t g = 8 * (int64_t)kXcdRun;
  return (unsigned)(((blocks + g - 1) / g) * g);
}

// A barrier for LDS accesses alone: global loads and atomics in flight stay in flight, where
// __syncthreads waits for them too.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ---- launches (each file defines its own) ----
hipError_t launch_preprocess(const PreParams &p, const PreOut &o, hipStream_t s);
// Scans of per-workgroup counts, one workgroup each.
struct ScanJob {
  const uint32_t *in;
  unsigned long long *prefix;
  uint32_t *total;
  unsigned long long *host_out;   // may be null
  int blocks;
};
struct ScanJobs {
  ScanJob job[FLOD_MAX_LEVELS];
};
hipError_t launch_scan_blocks(const ScanJobs &jobs, int n_jobs, uint32_t host_seq, hipStream_t s,
                              const unsigned long long *extra = nullptr);
int radix_items(int64_t n_max);        // keys per thread the radix sort of n_max keys uses
size_t radix_hist_bytes(int64_t n_max, bool depth = false);  // bytes of each of its hist and scan arrays
// The render's depth sort: the first pass reads keys[0, n_max) of every candidate, takes each
// key's index as its value and skips keys equal to kDepthNone (it writes the count it kept to
// *n_ptr, which the later passes read), its digit scan also takes the frame's totals, and the
// last pass also writes rect_out[pos] = rect_of[sorted value].
struct DepthSort {
  const uint32_t *keys;
  const uint2 *rect_of;
  uint2 *rect_out;
  const uint4 *sums;      // the preprocess's counts per workgroup
  uint4 *part;            // as many words of scratch: their sums per sort workgroup
  FrameTotals totals;     // its sums and nb are set to part's
  bool far;               // some depth may be 8192 or more
};
// The same for n <= kSmallSort candidates in one launch; blocks: the preprocess's workgroups.
hipError_t launch_depth_sort_small(const DepthSort &d, int64_t n, int blocks, uint32_t *vals_out, hipStream_t s);
hipError_t launch_radix_sort(uint32_t *keys[2], uint32_t *vals[2], uint32_t *n_ptr,
                             int64_t n_max, int bits, uint32_t *hist, uint32_t *scan,
                             uint32_t *tot, int *result_buf, hipStream_t s, const DepthSort *depth = nullptr);
// Exclusive prefix of each of `rows` rows of ceil(*n_ptr / tile) counts (scan may be hist), and the
// rows' sums.
hipError_t launch_row_scan(const uint32_t *n_ptr, const uint32_t *hist, uint32_t *scan, uint32_t *tot, int rows,
                           int stride, int tile, hipStream_t s);
// Binning through supertiles (tilebin.hip)
int super_count(const DevCamera &cam);
size_t pair_hist_bytes(const DevCamera &cam, int64_t n);       // bytes of its scan array
size_t pair_tot_bytes(const DevCamera &cam);                   // and of its tot array
int64_t chunk_capacity(const DevCamera &cam, int64_t pairs);   // the most chunks that many pairs make
hipError_t launch_pair_offsets(const uint32_t *ids, const uint32_t *counters, const uint2 *srect, const BinIn &bin,
                               const DevCamera &cam, int64_t n, uint32_t *scan, uint32_t *tot, hipStream_t s);
hipError_t launch_pair_place(const uint32_t *ids, uint32_t *counters, const uint2 *srect, const BinIn &bin,
                             const DevCamera &cam, int64_t n, const uint32_t *scan, uint32_t *tot,
                             uint32_t *pair_id, unsigned long long *pair_mask, uint4 *chunks, uint2 *supers,
                             hipStream_t s);
hipError_t launch_chunk_counts(const uint32_t *counters, const uint4 *chunks, const unsigned long long *pair_mask,
                               const uint2 *supers, const DevCamera &cam, int64_t max_chunks, uint32_t *cnt,
                               uint32_t *tile_len, hipStream_t s);
hipError_t launch_tile_starts(const uint32_t *tile_len, int n_tiles, uint2 *ranges, hipStream_t s);
hipError_t launch_chunk_expand(const uint32_t *counters, const uint4 *chunks, const uint32_t *pair_id,
                               const unsigned long long *pair_mask, const uint32_t *prefix, const uint2 *ranges,
                               const DevCamera &cam, int64_t max_chunks, uint32_t *values, const uint32_t *tile_len,
                               uint32_t *order, hipStream_t s);
hipError_t launch_frame_totals(const FrameTotals &t, hipStream_t s);
hipError_t launch_bin_records(int64_t n, const uint32_t *tiles, const uint2 *rect, const BinIn &in, float4 *out,
                              hipStream_t s);
hipError_t launch_tile_ids(const uint2 *ranges, int n_tiles, uint32_t *tile_ids, hipStream_t s);
// [start, end) of every bucket (id >> shift) in the sorted ids (ranges zeroed beforehand)
hipError_t launch_ranges(const uint32_t *ids, int shift, const uint32_t *k_ptr, int64_t k_max, uint2 *ranges,
                         hipStream_t s);
// blended: per tile, the (list position, Gaussian) pairs of the entries the forward blended
// into some pixel, in list order at the start of the tile's range; tile_blended: their count
// (both may be null: the render keeps no backward state)
hipError_t launch_blend(const uint2 *ranges, const uint32_t *values, const float4 *xyab,
                        const float4 *cop, const float2 *blue, const DevCamera &cam,
                        const float bg[3], float *image, float *final_T, int32_t *n_contrib,
                        int32_t *n_blended, uint2 *blended, uint32_t *tile_blended, const uint32_t *order,
                        hipStream_t s);
// order: n_tiles + 2 words of scratch (the backward's tile order and its counts of split tiles);
// g2d: the n_g2d gradient sums, doubles where bwd_sums_wide, else floats, zeroed here first; the kernel
// is timed by the events (if given), its tile order and the zeroing are not
hipError_t launch_blend_bwd(const uint2 *ranges, const float4 *xyab, const float4 *cop, const float2 *blue,
                            const DevCamera &cam, const float bg[3], const float *final_T,
                            const int32_t *n_contrib, const float *dL_dimage, void *g2d, int64_t n_g2d,
                            const uint2 *blended, const uint32_t *tile_blended, uint32_t *order,
                            hipStream_t s, hipEvent_t ev_start = nullptr, hipEvent_t ev_stop = nullptr);
// whether the backward of a frame of that many tiles adds its gradient sums in FP64
bool bwd_sums_wide(int n_tiles);
// the most blocks the backward's split tiles add beyond one per tile
int bwd_split_extra(int n_tiles);
// The blend backward's per-Gaussian moment sums (doubles when wide) into dL/d(mu', conic, opacity)
// and the colour's, as floats, to g2d (inspection; floats in place).
hipError_t launch_g2d_from_moments(int64_t n, const uint32_t *tiles, const float4 *xyab, const float4 *cop,
                                   const void *sums, bool wide, float *g2d, hipStream_t s);
// shjac: the forward preprocess's Jacobians and pre-clamp colours (PreOut::shjac)
// (g2d: doubles when wide)
hipError_t launch_preprocess_bwd(const PreParams &p, const uint32_t *tiles, const void *g2d, bool wide,
                                 const float4 *shjac, const flod_grads &g, hipStream_t s);
hipError_t launch_fill_u32(uint32_t *p, uint32_t v, int64_t n, hipStream_t s);
// The kept Gaussians of several levels' bands, counted per workgroup: level k's workgroups are
// first[k] .. first[k + 1] - 1 of the launch and of block_cnt.
struct BandCounts {
  const float *means[FLOD_MAX_LEVELS];
  int64_t n[FLOD_MAX_LEVELS];
  float lo2[FLOD_MAX_LEVELS], hi2[FLOD_MAX_LEVELS];
  int64_t first[FLOD_MAX_LEVELS + 1];
  float centre[3];
  int levels;
};
hipError_t launch_select_count(const BandCounts &c, uint32_t *block_cnt, hipStream_t s);
hipError_t launch_select_copy(const flod_level &in, const float centre[3], float lo2, float hi2,
                              const unsigned long long *prefix, const flod_level &out, hipStream_t s);
hipError_t launch_mask_count(const uint8_t *mask, int64_t n, uint32_t *block_cnt, hipStream_t s);
hipError_t launch_mask_copy(const flod_level &in, const uint8_t *mask, const unsigned long long *prefix,
                            const flod_level &out, hipStream_t s);
hipError_t launch_level_transition(const flod_level &in, float s_min_next, const flod_level &out, hipStream_t s);
hipError_t launch_adam(const AdamArgs &a, hipStream_t s);
int64_t ssim_blocks(int C, int H, int W);   // workgroups (and loss partials) of the SSIM kernels
hipError_t launch_ssim_forward(const float *x, const float *y, int C, int H, int W, float lam, double *loss,
                               float *gmap, double2 *partials, hipStream_t s);
hipError_t launch_ssim_backward(const float *x, const float *y, int C, int H, int W, float lam, const float *gmap,
                                const double *dloss, float *dx, hipStream_t s);
int64_t l1_blocks();   // workgroups (and loss partials) of the L1 forward
hipError_t launch_l1_forward(const float *x, const float *y, int64_t n, double *loss, double2 *partials,
                             hipStream_t s);
hipError_t launch_l1_backward(const float *x, const float *y, int64_t n, const double *dloss, float *dx,
                              hipStream_t s);
int prune_table_bits(int64_t n);   // log2 of the overlap-pruning hash table size for n points
int prune_levels(int64_t n);       // halvings of a cell its sort keys hold (3 bits each below the bucket)
// ranges, tags: 2^prune_table_bits(n) slots each, cleared here with the counters the others use
hipError_t launch_prune_keys(const float *means, int64_t n, float d_op, uint32_t *keys, uint32_t *vals, uint2 *ranges,
                             uint32_t *tags, uint32_t *counters, hipStream_t s);
// sums: kDepthRadix words, cleared here
hipError_t launch_prune_gather(const float *means, const uint32_t *sorted_vals, int64_t n, float4 *pts,
                               unsigned long long *sums, hipStream_t s);
// around: per point in key order, the points in the 27 buckets around it (itself included); sums: parts of
// their sum, which the query writes to cost, and of the count of points with many
hipError_t launch_prune_cost(const float4 *pts, const uint2 *ranges, int64_t n, float d_op, uint32_t *around,
                             unsigned long long *sums, hipStream_t s);
// runs: as many slots as tags
hipError_t launch_prune_runs(const uint32_t *keys, const uint2 *ranges, int64_t n, float d_op, uint32_t *tags,
                             uint2 *runs, hipStream_t s);
hipError_t launch_prune_query(const float4 *pts, const uint2 *ranges, const uint32_t *tags, const uint2 *runs,
                              uint32_t *around, int64_t n, float d_op, const unsigned long long *sums,
                              unsigned long long *cost, uint8_t *keep, double *d_avg, hipStream_t s);

}  // namespace flod
