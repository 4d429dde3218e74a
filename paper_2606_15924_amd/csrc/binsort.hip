// Tile x depth binning, sort and per-tile ranges.
//
// The per-tile Gaussian lists must follow (tile, FP32 depth bits, Gaussian
// id) and hold only the (Gaussian, tile) pairs whose tile can composite: the
// tile lies in the Gaussian's 3-sigma rectangle and its pixel-centre
// rectangle meets the ellipse q(d) <= t of the stored centre and conic.
// Row by row that is an interval of columns (row_span, FP64 with a fixed
// operation order).  Rather than radix-sorting a 64-bit (tile, depth) key
// with an id for every pair, the Gaussians are put in (depth, id) order once
// (a 32-bit sort of n keys), and their row intervals, not the pairs, are
// partitioned by tile row: a record (id, first column, last column) stands
// for 4-5 pairs.  Each tile row's records, which are in depth order, are then
// expanded straight into the tiles' lists.
//
//   sort      (depth, id) order of the Gaussians with a non-empty rectangle:
//             LSD radix sort, the others dropped in its first pass (or, for
//             few Gaussians, ranks by counting)
//   count     a thread per depth position over its rectangle rows: the row
//             intervals that hold a valid tile, counted per strip (a tile row,
//             or 256 columns of one in wider grids) and block
//   strips    per strip, the prefix of the blocks' counts and the totals; then
//             the strips' first record, pair and block, and the pair count
//   rows      the records, written to their strip in depth order
//   hist      a workgroup per 512 records of one strip: pairs per column
//             (a difference array, two LDS atomics per record)
//   offsets   per strip, the prefix over its blocks of every column, from the
//             tile's first pair on; the tiles' ranges
//   place     a workgroup per 512 records again: each record's rank among
//             the earlier records covering the column (a bit mask per column
//             over the wave's 64 records), the id written to the list
//
// Sorting row records instead of pairs moves 8 bytes per 4-5 pairs through
// the partition and writes each pair once; the pair-wise form (emit keys, two
// radix passes with their histograms, find the tile boundaries) moved every
// pair six times.  300k Gaussians, 1296 x 840, 5.7M pairs: 216 -> 155 us; 1.5M
// Gaussians, 1600 x 1060, 42M pairs: 745 -> 450 us.
#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdint>

#include "scan.h"

namespace tgs {

// ------------------------------------------------------------------ scans
template <typename T>
__global__ void __launch_bounds__(kScanThreads) scan_reduce_kernel(const T* __restrict__ in, int64_t n,
                                                                  T* __restrict__ part) {
  const int64_t base = (int64_t)blockIdx.x * kScanTile;
  T s = 0;
  for (int k = 0; k < kScanItems; ++k) {
    const int64_t i = base + (int64_t)k * kScanThreads + threadIdx.x;
    if (i < n) s += in[i];
  }
  __shared__ T lds[kScanThreads / kWave];
  T total;
  block_exclusive_scan<kScanThreads, T>(s, lds, &total);
  if (threadIdx.x == 0) part[blockIdx.x] = total;
}

// Down-sweep of a block: its prefix is the sum of the earlier blocks' sums
// (each block adds them up itself, so the scan takes two launches).
template <typename T>
__global__ void __launch_bounds__(kScanThreads) scan_down_kernel(const T* __restrict__ in, int64_t n,
                                                                const T* __restrict__ part,
                                                                T* __restrict__ out) {
  __shared__ T lds[kScanThreads / kWave];
  T before = 0;
  for (int64_t b = threadIdx.x; b < (int64_t)blockIdx.x; b += kScanThreads) before += part[b];
  T block_pre;
  (void)block_exclusive_scan<kScanThreads, T>(before, lds, &block_pre);
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  T v[kScanItems];
  T s = 0;
  for (int k = 0; k < kScanItems; ++k) {
    const int64_t i = base + k;
    v[k] = i < n ? in[i] : 0;
    s += v[k];
  }
  T total;
  T run = block_pre + block_exclusive_scan<kScanThreads, T>(s, lds, &total);
  for (int k = 0; k < kScanItems; ++k) {
    const int64_t i = base + k;
    if (i < n) out[i] = run;
    run += v[k];
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == kScanThreads - 1) out[n] = run;
}

template <typename T>
__global__ void __launch_bounds__(64) set_kernel(T* __restrict__ p, T v) {
  if (threadIdx.x == 0) *p = v;
}

// out[0..n] = exclusive prefix of in[0..n) and the total.
template <typename T>
static void exclusive_scan(const T* in, T* out, int64_t n, T* partials, hipStream_t s) {
  const int64_t nb = scan_partials(n);
  if (nb == 0) {
    hipLaunchKernelGGL(set_kernel<T>, dim3(1), dim3(64), 0, s, out, (T)0);
    return;
  }
  hipLaunchKernelGGL(scan_reduce_kernel<T>, dim3((unsigned)nb), dim3(kScanThreads), 0, s, in, n, partials);
  hipLaunchKernelGGL(scan_down_kernel<T>, dim3((unsigned)nb), dim3(kScanThreads), 0, s, in, n, partials, out);
}

void exclusive_scan_u32(const uint32_t* in, uint32_t* out, int64_t n, uint32_t* partials, hipStream_t s) {
  exclusive_scan<uint32_t>(in, out, n, partials, s);
}

// ------------------------------------------------------------------ row spans
// Depth key of a Gaussian without pairs: above every finite positive depth bit pattern.
constexpr uint32_t kCulledKey = 0xffffffffu;

// Rectangles are clamped to the tile grid (projection already does so; the
// clamp keeps every index of the binning in bounds for any input).
__device__ __forceinline__ int4 clamp_rect(int4 r, int tiles_x, int tiles_y) {
  r.x = min(max(r.x, 0), tiles_x);
  r.z = min(max(r.z, r.x), tiles_x);
  r.y = min(max(r.y, 0), tiles_y);
  r.w = min(max(r.w, r.y), tiles_y);
  return r;
}

// What the row test needs of one Gaussian: the stored centre (integer part
// and fraction) and conic widened to FP64 (exact), and per-Gaussian terms of
// the ellipse q(d) = A dx^2 + 2 B dx dy + C dy^2 <= t: det = AC - B^2,
// its half-height ym = sqrt(t A / det), ys = B sqrt(t / (C det)) (the
// rightmost point of the ellipse sits at dy = -ys, the leftmost at +ys) and
// tA = t A.  pd = 0 for a conic that is not positive definite.
//
// The bound t is the Gaussian's own: alpha = o exp(-q/2) reaches alpha_min
// only where q <= 2 ln(o / alpha_min), so t = that plus 0.004 (alpha below
// alpha_min by 0.2 % past it, far above the FP32 error of the renderer's
// alpha), rounded up to a multiple of 1/64, and at most tau (the bound for
// o = 1).  A Gaussian with t <= 0 keeps no tile (ym < 0 empties every row).
// lia = ln(1 / alpha_min).
struct RowEllipse {
  double xi, xf, yi, yf, A, iA, B, det, ym, ys, tA;  // iA: 1 / A
  int pd;
};

// ceil(64 (2 (ln o + lia) + 0.004)): from the hardware's float logarithm (good
// to 1e-6 here) unless that lies within 2.5e-4 of an integer.
__device__ __forceinline__ double ellipse_steps(float of, double lia) {
#pragma clang fp contract(off)
  const double q = 64.0 * (2.0 * ((double)__builtin_amdgcn_logf(of) * 0.69314718055994531 + lia) + 0.004);
  const double c = ceil(q), f = c - q;
  if (f > 2.5e-4 && f < 1.0 - 2.5e-4) return c;
  return ceil(64.0 * (2.0 * (log((double)of) + lia) + 0.004));
}

__device__ __forceinline__ RowEllipse row_ellipse(float4 p0, float4 p1, double tau, double lia) {
#pragma clang fp contract(off)
  RowEllipse e;
  const double t = p1.w > 0.f ? fmin(tau, ellipse_steps(p1.w, lia) * (1.0 / 64.0)) : -1.0;
  e.xi = p0.x;
  e.yi = p0.y;
  e.xf = p0.z;
  e.yf = p0.w;
  // the record's conic is (a, beta, delta) with b = beta a, c = delta + beta b,
  // det = a c - b^2 = a delta
  e.A = p1.x;
  e.iA = 1.0 / e.A;
  e.B = (double)p1.y * e.A;
  const double C = (double)p1.z + (double)p1.y * e.B;
  e.det = e.A * (double)p1.z;
  e.pd = e.A > 0.0 && e.det > 0.0;
  e.ym = !e.pd ? 0.0 : (t > 0.0 ? sqrt((t * e.A) / e.det) : -1.0);
  e.ys = e.pd && t > 0.0 ? e.B * sqrt(t / (C * e.det)) : 0.0;
  e.tA = t * e.A;
  return e;
}

// sqrt(x) to a few parts in 1e14 (0 for 0): the hardware's estimate and one
// Newton step.  A denormal x may give 0 (its root is below 1e-150).
__device__ __forceinline__ double near_sqrt(double x) {
  const double r = __builtin_amdgcn_rsq(x), g = x * r, h = 0.5 * r;
  const double s = __builtin_fma(g, __builtin_fma(-h, g, 0.5), g);
  return x > 1e-300 ? s : 0.0;
}

// Kept columns [lo, hi] of tile row ty inside the rectangle columns
// [rx0, rx1) (lo > hi when none): the tiles whose pixel-centre column range
// meets the x-extent of the ellipse cut by the row's pixel-centre strip.
// The right boundary of the ellipse, x(dy) = (sqrt(tA - det dy^2) - B dy)/A,
// is concave, so the strip's rightmost point is at the ellipse's rightmost
// dy clamped to the strip (the leftmost likewise).  FP64, IEEE operations
// in a fixed order and no contraction: the decision is reproducible bit for
// bit by any implementation of the same order.
__device__ __forceinline__ void row_span(const RowEllipse& e, int ty, int rx0, int rx1, int& lo, int& hi) {
#pragma clang fp contract(off)
  if (!e.pd) {  // keeps the whole rectangle row
    lo = rx0;
    hi = rx1 - 1;
    return;
  }
  const double Y0 = ((double)(kTile * ty) - e.yi) - e.yf;
  const double Y1 = ((double)(kTile * ty + kTile - 1) - e.yi) - e.yf;
  const double ylo = fmax(Y0, -e.ym), yhi = fmin(Y1, e.ym);
  if (!(ylo <= yhi)) {
    lo = rx0;
    hi = rx0 - 1;
    return;
  }
  const double yr = fmin(fmax(-e.ys, ylo), yhi);
  const double yl = fmin(fmax(e.ys, ylo), yhi);
  const double Dr = fmax(0.0, e.tA - e.det * (yr * yr)), Dl = fmax(0.0, e.tA - e.det * (yl * yl));
  const double br = e.B * yr, bl = e.B * yl;
  double l, h;
  {
    // the columns from roots and quotients good to 1e-13, when no rounding of
    // the exact operations could cross a column
    const double sr = near_sqrt(Dr), sl = near_sqrt(Dl);
    const double tl = (((-sl - bl) * e.iA + e.xf) + e.xi - (double)(kTile - 1)) * (1.0 / kTile);
    const double th = (((sr - br) * e.iA + e.xf) + e.xi) * (1.0 / kTile);
    const double size = fmax(fmax((sr + fabs(br)) * fabs(e.iA), (sl + fabs(bl)) * fabs(e.iA)), fabs(e.xi));
    l = ceil(tl);
    h = floor(th);
    // distance of the nearest column: 1e-6 columns against errors below 1e-12 size / 16
    const double fl = l - tl, fh = th - h;
    const bool sure = size < 1e6 && fl > 1e-6 && fl < 1.0 - 1e-6 && fh > 1e-6 && fh < 1.0 - 1e-6;
    if (!sure) {
      const double xmax = (sqrt(Dr) - br) / e.A;
      const double xmin = (-sqrt(Dl) - bl) / e.A;
      const double PL = (xmin + e.xf) + e.xi, PR = (xmax + e.xf) + e.xi;  // image pixel coordinates
      l = ceil((PL - (double)(kTile - 1)) * (1.0 / kTile));
      h = floor(PR * (1.0 / kTile));
    }
  }
  lo = (int)fmin(fmax(l, (double)rx0), (double)rx1);
  hi = (int)fmin(fmax(h, (double)(rx0 - 1)), (double)(rx1 - 1));
}

// ------------------------------------------------------------------ depth sort
// Blocks of 256 threads x 8 keys, 256 digits.
constexpr int kSortThreads = 256;
constexpr int kSortWaves = kSortThreads / kWave;
constexpr int kDepthItems = 8;
constexpr int kDepthBlockKeys = kSortThreads * kDepthItems;
constexpr int kDepthDigits = 256;

__device__ __forceinline__ uint64_t lanes_below() {
  const int lane = lane_id();
  return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

// Lanes of the wave holding the same digit (inactive lanes excluded), found
// through LDS: each active lane clears its digit's mask word, ORs in its own
// lane bit and reads the word back.  The three LDS operations of one wave
// execute in order, so every read sees exactly the bits of the lanes that
// share the digit.  s_mask holds one word per digit, private to the wave.
__device__ __forceinline__ uint64_t digit_peers(uint32_t d, bool valid, uint64_t* s_mask) {
  uint64_t peers = 0ull;
  if (valid) {
    s_mask[d] = 0ull;
    __hip_atomic_fetch_or(&s_mask[d], 1ull << lane_id(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    peers = __hip_atomic_load(&s_mask[d], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  return peers;
}

// A view's depth sort.  The views of a step go through every kernel together,
// one per grid layer: the short launches (scans, counts) are latency-bound, so
// three views in one take about as long as one.
struct DepthArgs {
  const int4* rect;
  const float* depth;
  uint32_t n;
  int tiles_x, tiles_y;
  int stride;          // row stride of the digit tables
  uint32_t* keys[2];
  uint32_t* vals[2];
  uint32_t* hist;      // [256][stride]
  uint32_t* hoffs;
  uint32_t* dtot;      // [256]
  uint32_t* n_keyed;
  int4* rects;         // nullable
  uint32_t* part;      // few Gaussians: partial ranks
};
using DepthBatch = Batch<DepthArgs>;

// Depth key of Gaussian i: its depth bits when its rectangle holds a tile
// (below kCulledKey also for a NaN depth), else kCulledKey.
__device__ __forceinline__ uint32_t depth_key(int4 r, float depth) {
  if (!(r.z > r.x && r.w > r.y)) return kCulledKey;
  return min(__float_as_uint(depth), kCulledKey - 1u);
}

// The depth keys, the first pass's digit counts of every block (culled
// Gaussians left out), and, when rects is given, the clamped rectangles (a
// depth-prefix call keeps them for its continuation).
__global__ void __launch_bounds__(kSortThreads) key_kernel(DepthBatch batch) {
  const DepthArgs& a = batch.v[blockIdx.z];
  __shared__ uint32_t h[kDepthDigits];
  h[threadIdx.x] = 0u;
  __syncthreads();
  const int64_t b0 = (int64_t)blockIdx.x * kDepthBlockKeys;
#pragma unroll
  for (int k = 0; k < kDepthItems; ++k) {
    const int64_t i = b0 + k * kSortThreads + threadIdx.x;
    if (i >= (int64_t)a.n) continue;
    const int4 r = clamp_rect(a.rect[i], a.tiles_x, a.tiles_y);
    const uint32_t key = depth_key(r, a.depth[i]);
    a.keys[0][i] = key;
    if (a.rects != nullptr) a.rects[i] = r;
    if (key != kCulledKey) atomicAdd(&h[key & (kDepthDigits - 1u)], 1u);
  }
  __syncthreads();
  a.hist[(int64_t)threadIdx.x * a.stride + blockIdx.x] = h[threadIdx.x];
}

// Digit counts of every block of the later passes (over the *n keys left).
__global__ void __launch_bounds__(kSortThreads) depth_hist_kernel(DepthBatch batch, int pass) {
  const DepthArgs& a = batch.v[blockIdx.z];
  const uint32_t* const keys = a.keys[pass & 1];
  const uint32_t n = *a.n_keyed;
  const int shift = 8 * pass;
  const int64_t b0 = (int64_t)blockIdx.x * kDepthBlockKeys;
  if (b0 >= (int64_t)n) return;  // the scan and the scatter stop at the last block that holds keys
  __shared__ uint32_t h[kDepthDigits];
  h[threadIdx.x] = 0u;
  uint32_t key[kDepthItems];
#pragma unroll
  for (int k = 0; k < kDepthItems; ++k) {
    const int64_t i = b0 + k * kSortThreads + threadIdx.x;
    key[k] = i < (int64_t)n ? keys[i] : 0u;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kDepthItems; ++k)
    if (b0 + k * kSortThreads + threadIdx.x < (int64_t)n)
      atomicAdd(&h[(key[k] >> shift) & (kDepthDigits - 1u)], 1u);
  __syncthreads();
  a.hist[(int64_t)threadIdx.x * a.stride + blockIdx.x] = h[threadIdx.x];
}

// One workgroup per digit: exclusive prefix of the digit's per-block counts
// (a contiguous row of the digit-major table) and the digit's total.  Only the
// blocks that hold keys have table entries.
__global__ void __launch_bounds__(1024) digit_scan_kernel(DepthBatch batch, int pass) {
  const DepthArgs& a = batch.v[blockIdx.z];
  __shared__ uint32_t lds[1024 / kWave];
  const int64_t n = pass == 0 ? a.n : *a.n_keyed;
  const int nblocks = (int)ceil_div(n, kDepthBlockKeys);
  const int64_t row = (int64_t)blockIdx.x * a.stride;
  uint32_t carry = 0;
  for (int b0 = 0; b0 < nblocks; b0 += 1024) {
    const int b = b0 + (int)threadIdx.x;
    const uint32_t v = b < nblocks ? a.hist[row + b] : 0u;
    uint32_t tot;
    const uint32_t ex = block_exclusive_scan<1024, uint32_t>(v, lds, &tot);
    if (b < nblocks) a.hoffs[row + b] = carry + ex;
    carry += tot;
  }
  if (threadIdx.x == 0) a.dtot[blockIdx.x] = carry;
}

// One pass of the depth sort: ranks a block's keys by digit (stable: by wave,
// round, lane), reorders them in LDS and writes runs of equal digits to
// consecutive addresses.  kFirst: the ids are the indices, culled keys are
// left out and the number kept goes to *n_keyed, which the later passes read.
// kLast: only the ids are written.
template <bool kFirst, bool kLast>
__global__ void __launch_bounds__(kSortThreads) depth_pass_kernel(DepthBatch batch, int pass) {
  const DepthArgs& a = batch.v[blockIdx.z];
  const uint32_t* const keys_in = a.keys[pass & 1];
  const uint32_t* const vals_in = a.vals[pass & 1];
  uint32_t* const keys_out = a.keys[(pass & 1) ^ 1];
  uint32_t* const vals_out = a.vals[(pass & 1) ^ 1];
  const int shift = 8 * pass;
  constexpr int kItems = kDepthItems, kBlockKeys = kDepthBlockKeys, kDigits = kDepthDigits;
  __shared__ uint32_t s_cnt[kSortWaves][kDigits];  // per-wave digit counts, then block-local offsets
  __shared__ uint32_t s_gbase[kDigits];            // global position of block-local position 0 of the digit
  __shared__ uint32_t s_keys[kBlockKeys];
  __shared__ uint32_t s_vals[kBlockKeys];
  __shared__ uint32_t s_red[kSortWaves];
  __shared__ uint64_t s_mask[kSortWaves][kDigits];
  const uint32_t n = kFirst ? a.n : *a.n_keyed;
  const int64_t blk0 = (int64_t)blockIdx.x * kBlockKeys;
  if (blk0 >= (int64_t)n) return;  // workgroup-uniform
  const int tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
  for (int i = tid; i < kSortWaves * kDigits; i += kSortThreads) (&s_cnt[0][0])[i] = 0;
  // keys of digit tid in the earlier blocks, and in all blocks
  const uint32_t before = a.hoffs[(int64_t)tid * a.stride + blockIdx.x], all_d = a.dtot[tid];
  const int64_t wbase = blk0 + (int64_t)wave * kWave * kItems;
  uint32_t key[kItems], val[kItems];
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    const int64_t i = wbase + k * kWave + lane;
    key[k] = i < n ? keys_in[i] : kCulledKey;
    val[k] = kFirst ? (uint32_t)i : (i < n ? vals_in[i] : 0u);
  }
  auto have = [&](int k) { return kFirst ? key[k] != kCulledKey : wbase + k * kWave + lane < n; };
  __syncthreads();
  const uint64_t below = lanes_below();
  uint32_t rank[kItems];
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    const bool valid = have(k);
    const uint32_t d = (key[k] >> shift) & (kDigits - 1u);
    const uint64_t peers = digit_peers(d, valid, s_mask[wave]);
    const uint32_t r = (uint32_t)__popcll(peers & below);
    const uint32_t prior = valid ? s_cnt[wave][d] : 0u;
    rank[k] = prior + r;
    if (valid && r == 0) s_cnt[wave][d] = prior + (uint32_t)__popcll(peers);
  }
  __syncthreads();
  uint32_t pre[kSortWaves];
  uint32_t tot = 0;
  for (int w = 0; w < kSortWaves; ++w) {
    pre[w] = tot;
    tot += s_cnt[w][tid];
  }
  uint32_t count, all;
  const uint32_t lstart = block_exclusive_scan<kSortThreads, uint32_t>(tot, s_red, &count);
  const uint32_t dstart = block_exclusive_scan<kSortThreads, uint32_t>(all_d, s_red, &all);
  for (int w = 0; w < kSortWaves; ++w) s_cnt[w][tid] = lstart + pre[w];
  s_gbase[tid] = dstart + before - lstart;
  if (kFirst && blockIdx.x == 0 && tid == 0) *a.n_keyed = all;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    if (have(k)) {
      const uint32_t d = (key[k] >> shift) & (kDigits - 1u);
      const uint32_t lp = s_cnt[wave][d] + rank[k];
      if (lp < (uint32_t)kBlockKeys) {  // always (ranks are a permutation); a safeguard
        s_keys[lp] = key[k];
        s_vals[lp] = val[k];
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    const uint32_t lp = (uint32_t)(k * kSortThreads + tid);
    if (lp < count) {
      const uint32_t kk = s_keys[lp];
      const uint32_t dst = s_gbase[(kk >> shift) & (kDigits - 1u)] + lp;
      if (dst >= a.n) continue;  // never taken for a consistent table; keeps every write in bounds
      if (!kLast) keys_out[dst] = kk;
      vals_out[dst] = s_vals[lp];
    }
  }
}

// Few Gaussians: the rank of every key by counting the keys before it.  The
// twelve launches above take ~5 us each whatever n is (57 us in all); n^2
// comparisons spread over the chip take 18 us at 10,000 Gaussians, a sort
// in one workgroup's LDS 47 us.  Whole calls on 256 x 256 images, ranks and
// passes: one view of 10,000 Gaussians 58 and 100 us, 16,384 66 and 100, 24,000
// 89 and 102, 28,000 104 and 104; four views in one call, which share the
// passes' latency but not the comparisons, 10,000 79 and 109, 16,384 114 and 110,
// 20,000 160 and 111.  The line lies where four views break even.
//
// rank: 256 Gaussians against 256 others per workgroup.  Keys tie-break by
// index, so a chunk of others before the workgroup's Gaussians counts its
// equal keys and one after them does not; only the chunk holding them compares
// the indices.
constexpr int64_t kSmallSort = 16384;
constexpr int kRankThreads = 256;
constexpr int kRankChunk = kRankThreads;

__global__ void __launch_bounds__(kRankThreads) rank_kernel(DepthBatch batch) {
  const DepthArgs& a = batch.v[blockIdx.z];
  const uint32_t n = a.n;
  __shared__ __align__(16) uint32_t s_key[kRankChunk];
  __shared__ uint32_t s_kept;
  const int tid = threadIdx.x;
  const uint32_t i = blockIdx.x * (uint32_t)kRankThreads + tid, j0 = blockIdx.y * (uint32_t)kRankChunk;
  if (tid == 0) s_kept = 0u;
  __syncthreads();
  {
    const uint32_t j = j0 + tid;
    uint32_t other = kCulledKey;  // past the end: before no key
    if (j < n) other = depth_key(clamp_rect(a.rect[j], a.tiles_x, a.tiles_y), a.depth[j]);
    s_key[tid] = other;
    const uint64_t have = ballot(other != kCulledKey);
    if (blockIdx.x == 0 && lane_id() == 0) atomicAdd(&s_kept, (uint32_t)__popcll(have));
  }
  uint32_t key = kCulledKey;
  if (i < n) {
    const int4 r = clamp_rect(a.rect[i], a.tiles_x, a.tiles_y);
    key = depth_key(r, a.depth[i]);
    if (a.rects != nullptr && blockIdx.y == 0) a.rects[i] = r;
  }
  __syncthreads();
  uint32_t rank = 0;
  const uint4* const k4 = reinterpret_cast<const uint4*>(s_key);
  // workgroup-uniform branches
  if (blockIdx.y < blockIdx.x) {
#pragma unroll 8
    for (int q = 0; q < kRankChunk / 4; ++q) {
      const uint4 o = k4[q];
      rank += (o.x <= key ? 1u : 0u) + (o.y <= key ? 1u : 0u) + (o.z <= key ? 1u : 0u) + (o.w <= key ? 1u : 0u);
    }
  } else if (blockIdx.y > blockIdx.x) {
#pragma unroll 8
    for (int q = 0; q < kRankChunk / 4; ++q) {
      const uint4 o = k4[q];
      rank += (o.x < key ? 1u : 0u) + (o.y < key ? 1u : 0u) + (o.z < key ? 1u : 0u) + (o.w < key ? 1u : 0u);
    }
  } else {
#pragma unroll 8
    for (int q = 0; q < kRankChunk / 4; ++q) {
      const uint4 o = k4[q];
      const int l = tid - 4 * q;  // others before this Gaussian: o.x for l > 0, o.y for l > 1, ...
      rank += (l > 0 ? o.x <= key : o.x < key) ? 1u : 0u;
      rank += (l > 1 ? o.y <= key : o.y < key) ? 1u : 0u;
      rank += (l > 2 ? o.z <= key : o.z < key) ? 1u : 0u;
      rank += (l > 3 ? o.w <= key : o.w < key) ? 1u : 0u;
    }
  }
  if (i < n) a.part[(int64_t)blockIdx.y * n + i] = key == kCulledKey ? ~0u : rank;
  if (blockIdx.x == 0 && tid == 0) a.dtot[blockIdx.y] = s_kept;
}

__global__ void __launch_bounds__(kRankThreads) rank_place_kernel(DepthBatch batch, int chunks) {
  const DepthArgs& a = batch.v[blockIdx.z];
  const uint32_t n = a.n, i = blockIdx.x * (uint32_t)kRankThreads + threadIdx.x;
  if (i < n && a.part[i] != ~0u) {
    uint32_t r = 0;
#pragma unroll 8
    for (int c = 0; c < chunks; ++c) r += a.part[(int64_t)c * n + i];
    if (r < n) a.vals[0][r] = i;  // always (the ranks are a permutation); a safeguard
  }
  if (i == 0) {
    uint32_t t = 0;
    for (int c = 0; c < chunks; ++c) t += a.dtot[c];
    *a.n_keyed = t;
  }
}

// ------------------------------------------------------------------ valid tiles
// Set bits of the columns [lo, hi] of a row of bits.
__device__ __forceinline__ uint32_t valid_in(const uint64_t* __restrict__ row, int lo, int hi) {
  uint32_t c = 0;
  for (int w = lo >> 6; lo <= hi && w <= hi >> 6; ++w) {
    uint64_t b = row[w];
    if (w == lo >> 6) b &= ~0ull << (lo & 63);
    if (w == hi >> 6) b &= ~0ull >> (63 - (hi & 63));
    c += (uint32_t)__popcll(b);
  }
  return c;
}

// ------------------------------------------------------------------ row records
// Strips: a tile row, cut into pieces of kStripCols columns when it has more
// (strip (y, c) holds the tiles of row y with x / kStripCols = c), in tile
// order.  The count keeps two counters per strip in LDS and a table entry per
// strip and block, so grids of more strips than a group holds are taken in
// groups, one after the other, each counted again before its records and with
// the rows of other groups left out.  The records need 24 times a counter's LDS:
// a workgroup writes those of kSub strips.  Groups of kSub throughout made the
// 272 rows of a 512 x 4352 image two groups and the 512 x 2 strips of 8192 x
// 8192 four: 300k Gaussians 608 -> 243 us and 10k 1505 -> 245 us with one.
constexpr int kStripCols = 256;  // a record's columns within its strip are 8 bits each
constexpr int kSub = 256;
constexpr int kRowThreads = 256;  // depth positions per block of the row stages
constexpr int kRowWaves = kRowThreads / kWave;
// The count keeps the intervals of a block's first rows for the records, which
// evaluate the others again: 36 rows per position, the most whose LDS leaves the
// workgroups that the registers allow, or 24 (48 bytes per Gaussian) for many
// Gaussians.  Few Gaussians, whose tables are small, also take larger groups.
// 30k of 45 rows on average, 300 x 1920: 175 us, with 24 rows 205; 100k of 12,
// 3840 x 2160: 234 us, with 12 rows 293; 10k in the 4096 strips of 16384 x
// 16384: 201 us in one group, 468 in four.
constexpr int64_t kFewGaussians = 1 << 17;
constexpr int kSpans = 24 * kRowThreads, kSpansFew = 36 * kRowThreads;
constexpr int kGroup = 1024, kGroupFew = 4096;
constexpr int kRecThreads = 256;
constexpr int kRecItems = 2;
constexpr int kRecBlock = kRecThreads * kRecItems;  // records per block of the pair stages

struct BinArgs {
  const uint32_t* n_keyed;    // Gaussians in the depth order (device)
  int64_t pos0, pos_end;      // the depth positions taken: [pos0, min(pos_end, *n_keyed))
  const uint32_t* ids;        // Gaussians in depth order
  const int4* rect;           // by Gaussian
  const float4* splat;
  uint64_t* bits;             // valid tiles (nullptr: all)
  const uint32_t* n_flagged;  // nullable: nothing is listed when it is 0
  int tiles_x, tiles_y, wpr;
  int sc;                     // strips per tile row
  int s0, sn;                 // the group: strips [s0, s0 + sn)
  int y0, y1;                 // its tile rows
  int group;                  // strips in a group
  double tau, lia;
  int64_t kb;                 // blocks of depth positions: row stride of the tables
  int span_rows;              // rows of a block whose intervals are kept
  uint32_t* rows_tab;         // [sn][kb] records per strip and block, then their prefix
  uint32_t* pairs_tab;        // [sn][kb] pairs
  uint16_t* spans;            // [blocks][span_rows] the block's rows' intervals, position after position
  int2* rowinfo;              // [positions] first tile row, rows
  uint8_t* touched;
  // per strip (all groups)
  unsigned long long* row_tot;
  unsigned long long* pair_tot;
  uint32_t* row_base;         // [S + 1]
  uint32_t* pair_base;
  uint32_t* blk_base;
  uint32_t* eff_total;        // all pairs when they fit the capacity, else 0
  uint2* rec;                 // [capacity] records: id, first column | last column << 8
  uint32_t* hist;             // [blocks of the group][cols] pairs per column, then first list positions
  int cols;                   // its row length: columns per strip
  uint32_t* vals;
  uint64_t* keys64;           // nullable
  const float* depth;         // for keys64
  uint2* ranges;
  const int32_t* tile_slot;   // nullable: the bits are made from it
  int64_t m, capacity;        // m >= 0: a depth-prefix call over m positions
  unsigned long long* counts; // the call's counts in its workspace
  unsigned long long* out;    // nullable: the caller's
  bool counted;               // the tables hold the counts (of one group of strips)
};
using BinBatch = Batch<BinArgs>;

// One bit per tile, wpr 64-bit words per tile row: the tiles whose map entry
// is >= 0.  A wave per row.
__global__ void __launch_bounds__(kWave) tile_bits_kernel(BinBatch batch) {
  const BinArgs& a = batch.v[blockIdx.z];
  const int64_t y = blockIdx.x;
  if (a.tile_slot == nullptr || y >= a.tiles_y) return;
  for (int w = 0; w < a.wpr; ++w) {
    const int x = w * kWave + lane_id();
    const uint64_t b = ballot(x < a.tiles_x && a.tile_slot[y * a.tiles_x + x] >= 0);
    if (lane_id() == 0) a.bits[y * a.wpr + w] = b;
  }
}

__device__ __forceinline__ int64_t bin_end(const BinArgs& a) { return min(a.pos_end, (int64_t)*a.n_keyed); }
__device__ __forceinline__ bool bin_nothing(const BinArgs& a) { return a.n_flagged != nullptr && *a.n_flagged == 0u; }

// Kept tiles of row ty, a piece per strip of the group: f(strip in the group,
// first column, last column, valid tiles) for each piece with a valid tile.
template <bool kWide, typename F>
__device__ __forceinline__ void row_pieces(const BinArgs& a, int ty, int lo, int hi, F&& f) {
  if (lo > hi) return;
  const uint64_t* brow = a.bits != nullptr ? a.bits + (int64_t)ty * a.wpr : nullptr;
  if (!kWide) {
    const uint32_t c = brow != nullptr ? valid_in(brow, lo, hi) : (uint32_t)(hi - lo + 1);
    if (c > 0) f(ty - a.s0, lo, hi, c);
    return;
  }
  for (int q = lo / kStripCols; q <= hi / kStripCols; ++q) {
    const int l = max(lo, q * kStripCols), h = min(hi, q * kStripCols + kStripCols - 1);
    const uint32_t c = brow != nullptr ? valid_in(brow, l, h) : (uint32_t)(h - l + 1);
    if (c > 0) f((int)((int64_t)ty * a.sc + q - a.s0), l - q * kStripCols, h - q * kStripCols, c);
  }
}

// The rows of the rectangle that the ellipse can meet: rows of pixel centres
// 16 ty .. 16 ty + 15 with 16 ty + 15 >= cy - ym and 16 ty <= cy + ym, widened
// by far more than FP64 rounds (row_span decides; this only saves it the rows
// past the ellipse, two of seven on average).
__device__ __forceinline__ void ellipse_rows(const RowEllipse& e, int4 r, int& y0, int& y1) {
  y0 = r.y;
  y1 = r.w;
  if (!e.pd) return;
  const double cy = e.yi + e.yf, eps = 1e-9 * (fabs(cy) + e.ym) + 1e-6;
  const double f = ceil((cy - e.ym - (double)(kTile - 1) - eps) * (1.0 / kTile));
  const double l = floor((cy + e.ym + eps) * (1.0 / kTile));
  y0 = (int)fmin(fmax(f, (double)r.y), (double)r.w);
  y1 = (int)fmin(fmax(l + 1.0, (double)y0), (double)r.w);
}

// Rows k and on of the few lanes that have them go to the wave, a Gaussian's
// rows one per lane, when handing a Gaussian over (~1.5 rows' work) costs less
// than walking to the longest.
__device__ __forceinline__ bool few_long(int rows, int k, int longest) {
  return 3 * __builtin_popcountll(ballot(rows > k)) <= 2 * (longest - k);
}

__device__ __forceinline__ double lane_f64(double v, int l) {
  return __longlong_as_double((long long)readlane_u64((uint64_t)__double_as_longlong(v), l));
}

__device__ __forceinline__ RowEllipse ellipse_of_lane(const RowEllipse& e, int l) {
  return {lane_f64(e.xi, l), lane_f64(e.xf, l),  lane_f64(e.yi, l), lane_f64(e.yf, l),
          lane_f64(e.A, l),  lane_f64(e.iA, l),  lane_f64(e.B, l),  lane_f64(e.det, l),
          lane_f64(e.ym, l), lane_f64(e.ys, l),  lane_f64(e.tA, l), __builtin_amdgcn_readlane(e.pd, l)};
}

// Count.  Bound by the gathers in depth order: at 1.5M Gaussians and 42M pairs,
// rectangle and tables take 31 us, the records 29 and the rows 32 (92 us; with
// IEEE roots and quotients in every row and without the shared walk 105 us).
// Handing the rows of 64 Gaussians out one per lane keeps every lane busy, but
// costs a prefix sum, two exchanges through LDS and their barriers per 64
// rows, which took longer than the idle lanes do.
template <bool kWide>
__global__ void __launch_bounds__(kRowThreads, 6) bin_count_kernel(BinBatch batch) {
  const BinArgs& a = batch.v[blockIdx.z];
  extern __shared__ uint32_t s_dyn[];  // two counters per strip, then the kept rows' intervals
  uint32_t* const s_rows = s_dyn;
  uint32_t* const s_pairs = s_dyn + a.sn;
  uint16_t* const s_span = reinterpret_cast<uint16_t*>(s_dyn + 2 * a.sn);
  __shared__ uint32_t s_red[kRowWaves];
  if (bin_nothing(a)) return;
  const int tid = threadIdx.x;
  const int64_t end = bin_end(a), p0 = a.pos0 + (int64_t)blockIdx.x * kRowThreads, p = p0 + tid;
  if (p0 >= end) return;  // workgroup-uniform
  for (int i = tid; i < a.sn; i += kRowThreads) {
    s_rows[i] = 0u;
    s_pairs[i] = 0u;
  }
  int4 r = make_int4(0, 0, 0, 0);
  float4 c0 = make_float4(0.f, 0.f, 0.f, 0.f), c1 = c0;
  uint32_t g = 0;
  if (p < end) {
    g = a.ids[p];
    r = clamp_rect(a.rect[g], a.tiles_x, a.tiles_y);
    r.y = max(r.y, a.y0);
    r.w = max(min(r.w, a.y1), r.y);
    if (a.bits == nullptr) {  // every listed Gaussian has a tile: its record is asked for beside the rectangle
      c0 = a.splat[3 * (int64_t)g];
      c1 = a.splat[3 * (int64_t)g + 1];
    }
  }
  bool some = r.z > r.x && r.w > r.y;
  if (a.bits != nullptr && some) {
    // a rectangle without a valid tile is done before its record is read
    some = false;
    for (int y = r.y; y < r.w && !some; ++y) some = valid_in(a.bits + (int64_t)y * a.wpr, r.x, r.z - 1) > 0;
  }
  RowEllipse e = {};
  int y0 = 0, y1 = 0;
  if (some) {
    if (a.bits != nullptr) {
      c0 = a.splat[3 * (int64_t)g];
      c1 = a.splat[3 * (int64_t)g + 1];
    }
    e = row_ellipse(c0, c1, a.tau, a.lia);
    ellipse_rows(e, r, y0, y1);
  }
  uint32_t total;
  const uint32_t at = block_exclusive_scan<kRowThreads, uint32_t>((uint32_t)(y1 - y0), s_red, &total);
  auto row = [&](const RowEllipse& re, int y, int rx0, int rx1, uint32_t q) {  // whether the row keeps a tile
    int lo, hi;
    row_span(re, y, rx0, rx1, lo, hi);
    uint32_t span = 0xffu;  // first column 255, last 0: empty
    bool kept = false;
    row_pieces<kWide>(a, y, lo, hi, [&](int s, int l, int h, uint32_t c) {
      kept = true;
      span = (uint32_t)l | ((uint32_t)h << 8);
      if (s >= 0 && s < a.sn) {
        atomicAdd(&s_rows[s], 1u);
        atomicAdd(&s_pairs[s], c);
      }
    });
    if (!kWide && q < (uint32_t)a.span_rows) s_span[q] = (uint16_t)span;
    return kept;
  };
  bool any = false;
  const int rows = y1 - y0, longest = wave_max_i(rows);
  int k = 0;
  for (; k < longest && !few_long(rows, k, longest); ++k)
    if (k < rows) any |= row(e, y0 + k, r.x, r.z, at + (uint32_t)k);
  for (uint64_t left = ballot(rows > k); left != 0ull; left &= left - 1) {
    const int l = (int)__builtin_ctzll(left);
    const RowEllipse el = ellipse_of_lane(e, l);
    const int n_l = __builtin_amdgcn_readlane(rows, l), y_l = __builtin_amdgcn_readlane(y0, l);
    const int rx0 = __builtin_amdgcn_readlane(r.x, l), rx1 = __builtin_amdgcn_readlane(r.z, l);
    const uint32_t at_l = (uint32_t)__builtin_amdgcn_readlane((int)at, l);
    bool kept = false;
    for (int j = k + lane_id(); j < n_l; j += kWave) kept |= row(el, y_l + j, rx0, rx1, at_l + (uint32_t)j);
    if (ballot(kept) != 0ull && lane_id() == l) any = true;
  }
  if (p < end) {
    if (any && a.touched != nullptr) a.touched[g] = 1;
    a.rowinfo[p - a.pos0] = make_int2(y0, y1 - y0);
  }
  __syncthreads();
  if (!kWide) {
    const uint32_t words = (min(total, (uint32_t)a.span_rows) + 1u) / 2u;
    uint32_t* dst = reinterpret_cast<uint32_t*>(a.spans + (int64_t)blockIdx.x * a.span_rows);
    for (uint32_t i = tid; i < words; i += kRowThreads) dst[i] = reinterpret_cast<const uint32_t*>(s_span)[i];
  }
  for (int i = tid; i < a.sn; i += kRowThreads) {
    a.rows_tab[(int64_t)i * a.kb + blockIdx.x] = s_rows[i];
    a.pairs_tab[(int64_t)i * a.kb + blockIdx.x] = s_pairs[i];
  }
}

// A workgroup per strip of the group: the prefix of its records over the
// blocks (in place), its records and its pairs.
__global__ void __launch_bounds__(1024) strip_scan_kernel(BinBatch batch) {
  const BinArgs& a = batch.v[blockIdx.z];
  if ((int)blockIdx.x >= a.sn) return;  // the grid is sized for the view of the most strips
  __shared__ uint32_t lds[1024 / kWave];
  __shared__ unsigned long long lds64[1024 / kWave];
  const int64_t end = bin_end(a);
  const int64_t nb = bin_nothing(a) || end <= a.pos0 ? 0 : ceil_div(end - a.pos0, kRowThreads);
  uint32_t* rows = a.rows_tab + (int64_t)blockIdx.x * a.kb;
  const uint32_t* pairs = a.pairs_tab + (int64_t)blockIdx.x * a.kb;
  unsigned long long np = 0;
  uint32_t carry = 0;
  for (int64_t b0 = 0; b0 < nb; b0 += 1024) {
    const int64_t b = b0 + threadIdx.x;
    const uint32_t v = b < nb ? rows[b] : 0u;
    if (b < nb) np += pairs[b];
    uint32_t tot;
    const uint32_t ex = block_exclusive_scan<1024, uint32_t>(v, lds, &tot);
    if (b < nb) rows[b] = carry + ex;
    carry += tot;
  }
  unsigned long long all;
  (void)block_exclusive_scan<1024, unsigned long long>(np, lds64, &all);
  if (threadIdx.x == 0) {
    a.row_tot[a.s0 + blockIdx.x] = carry;
    a.pair_tot[a.s0 + blockIdx.x] = all;
  }
}

// One workgroup: every strip's first record, pair and pair-stage block, and
// the counts.  out (nullable) receives counts[0] = counts[1] = pairs; with
// m >= 0 (a depth-prefix call over m positions) also an estimate of the whole
// lists' pairs: the prefix's pairs per Gaussian times the keyed Gaussians
// (exact when the prefix holds them all; the nearest Gaussians cover the most
// tiles, so it tends to exceed the count).
__global__ void __launch_bounds__(1024) strip_base_kernel(BinBatch batch) {
  const BinArgs& a = batch.v[blockIdx.z];
  const int64_t strips = (int64_t)a.sc * a.tiles_y;
  __shared__ unsigned long long lds[1024 / kWave];
  unsigned long long rows = 0, pairs = 0, blks = 0;  // before the strips of this round
  for (int64_t s0 = 0; s0 < strips; s0 += 1024) {
    const int64_t s = s0 + threadIdx.x;
    const unsigned long long r = s < strips ? a.row_tot[s] : 0ull, p = s < strips ? a.pair_tot[s] : 0ull;
    unsigned long long tr, tp, tb;
    const unsigned long long er = block_exclusive_scan<1024, unsigned long long>(r, lds, &tr);
    const unsigned long long ep = block_exclusive_scan<1024, unsigned long long>(p, lds, &tp);
    const unsigned long long eb =
        block_exclusive_scan<1024, unsigned long long>((r + kRecBlock - 1) / kRecBlock, lds, &tb);
    if (s < strips) {  // they wrap only past 2^32 pairs, where nothing reads them
      a.row_base[s] = (uint32_t)(rows + er);
      a.pair_base[s] = (uint32_t)(pairs + ep);
      a.blk_base[s] = (uint32_t)(blks + eb);
    }
    rows += tr;
    pairs += tp;
    blks += tb;
  }
  if (threadIdx.x == 0) {
    a.row_base[strips] = (uint32_t)rows;
    a.pair_base[strips] = (uint32_t)pairs;
    a.blk_base[strips] = (uint32_t)blks;
    a.counts[0] = pairs;
    a.counts[1] = pairs;
    *a.eff_total = pairs <= (unsigned long long)a.capacity ? (uint32_t)pairs : 0u;
    if (a.out != nullptr) {
      a.out[0] = pairs;
      a.out[1] = pairs;
      if (a.m >= 0) {
        const unsigned long long k = *a.n_keyed, mk = (unsigned long long)a.m < k ? (unsigned long long)a.m : k;
        a.out[2] = mk >= k || mk == 0 ? pairs : (unsigned long long)ceil((double)pairs * (double)k / (double)mk);
      }
    }
  }
}

// Records.  Per wave a 64-bit mask per strip collects which of its 64 depth
// positions have a record there; a record's place is the strip's first one,
// plus the earlier blocks', the earlier waves' and the earlier lanes' records.
template <bool kWide>
__global__ void __launch_bounds__(kRowThreads, 6) bin_rows_kernel(BinBatch batch) {
  const BinArgs& a = batch.v[blockIdx.z];
  __shared__ uint64_t s_mask[kRowWaves][kSub];
  __shared__ uint32_t s_pos[kRowWaves][kSub];
  extern __shared__ uint32_t s_dyn[];  // the kept rows' intervals
  uint16_t* const s_span = reinterpret_cast<uint16_t*>(s_dyn);
  __shared__ uint32_t s_red[kRowWaves];
  if (bin_nothing(a)) return;
  const int tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
  const int64_t end = bin_end(a), p0 = a.pos0 + (int64_t)blockIdx.x * kRowThreads, p = p0 + tid;
  const int t0 = (int)blockIdx.y * kSub, tn = min(kSub, a.sn - t0);  // strips of the group
  if (p0 >= end || *a.eff_total == 0u || tn <= 0) return;  // workgroup-uniform
  static_assert(kSub == kRowThreads, "a thread per strip");
#pragma unroll
  for (int w = 0; w < kRowWaves; ++w) s_mask[w][tid] = 0ull;
  int2 info = make_int2(0, 0);
  uint32_t g = 0;
  if (p < end) {
    info = a.rowinfo[p - a.pos0];
    g = a.ids[p];
  }
  uint32_t total;
  uint32_t at = block_exclusive_scan<kRowThreads, uint32_t>((uint32_t)info.y, s_red, &total);
  {
    // the rows that these strips are of
    const int s0 = a.s0 + t0, sc = kWide ? a.sc : 1, f = s0 / sc, l = (s0 + tn - 1) / sc + 1;
    const int skip = min(max(f - info.x, 0), info.y);
    at += (uint32_t)skip;
    info = make_int2(info.x + skip, max(min(info.y - skip, l - info.x - skip), 0));
  }
  if (!kWide) {
    const uint32_t words = (min(total, (uint32_t)a.span_rows) + 1u) / 2u;
    const uint32_t* src = reinterpret_cast<const uint32_t*>(a.spans + (int64_t)blockIdx.x * a.span_rows);
    for (uint32_t i = tid; i < words; i += kRowThreads) reinterpret_cast<uint32_t*>(s_span)[i] = src[i];
  }
  RowEllipse e = {};
  int4 r = make_int4(0, 0, 0, 0);
  if (info.y > 0 && (kWide || at + (uint32_t)info.y > (uint32_t)a.span_rows)) {  // rows not kept: evaluated again
    r = clamp_rect(a.rect[g], a.tiles_x, a.tiles_y);
    e = row_ellipse(a.splat[3 * (int64_t)g], a.splat[3 * (int64_t)g + 1], a.tau, a.lia);
  }
  __syncthreads();
  // f(strip of these, columns, lane whose row it is, its Gaussian)
  const int longest = wave_max_i(info.y);
  auto pieces = [&](const RowEllipse& re, int y, int rx0, int rx1, int l, uint32_t gl, auto&& f) {
    int lo, hi;
    row_span(re, y, rx0, rx1, lo, hi);
    row_pieces<kWide>(a, y, lo, hi, [&](int s, int x0, int x1, uint32_t) {
      if (s >= t0 && s < t0 + tn) f(s - t0, (uint32_t)x0 | ((uint32_t)x1 << 8), l, gl);
    });
  };
  auto stored = [&](int y, uint32_t q, int l, uint32_t gl, auto&& f) {
    const uint32_t c = s_span[q];
    const int s = y - a.s0 - t0;
    if ((c & 0xffu) <= (c >> 8) && s >= 0 && s < tn) f(s, c, l, gl);
  };
  const uint64_t kept = ballot(!kWide && at + (uint32_t)info.y <= (uint32_t)a.span_rows);
  auto each = [&](auto&& f) {
    int k = 0;
    for (; k < longest && !few_long(info.y, k, longest); ++k)
      if (k < info.y) {
        if (!kWide && at + (uint32_t)k < (uint32_t)a.span_rows) stored(info.x + k, at + (uint32_t)k, lane, g, f);
        else pieces(e, info.x + k, r.x, r.z, lane, g, f);
      }
    for (uint64_t left = ballot(info.y > k); left != 0ull; left &= left - 1) {
      const int l = (int)__builtin_ctzll(left);
      const int n_l = __builtin_amdgcn_readlane(info.y, l), y_l = __builtin_amdgcn_readlane(info.x, l);
      const uint32_t g_l = (uint32_t)__builtin_amdgcn_readlane((int)g, l);
      if (!kWide && (kept >> l) & 1ull) {
        const uint32_t at_l = (uint32_t)__builtin_amdgcn_readlane((int)at, l);
        for (int j = k + lane; j < n_l; j += kWave) stored(y_l + j, at_l + (uint32_t)j, l, g_l, f);
      } else {
        const RowEllipse el = ellipse_of_lane(e, l);
        const int rx0 = __builtin_amdgcn_readlane(r.x, l), rx1 = __builtin_amdgcn_readlane(r.z, l);
        for (int j = k + lane; j < n_l; j += kWave) pieces(el, y_l + j, rx0, rx1, l, g_l, f);
      }
    }
  };
  each([&](int s, uint32_t, int l, uint32_t) {
    __hip_atomic_fetch_or(&s_mask[wave][s], 1ull << l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  });
  __syncthreads();
  if (tid < tn) {
    uint32_t q = a.row_base[a.s0 + t0 + tid] + a.rows_tab[(int64_t)(t0 + tid) * a.kb + blockIdx.x];
#pragma unroll
    for (int w = 0; w < kRowWaves; ++w) {
      s_pos[w][tid] = q;
      q += (uint32_t)__popcll(s_mask[w][tid]);
    }
  }
  __syncthreads();
  const uint32_t rows_all = *a.eff_total;  // a record holds a pair, so there are no more records than pairs
  each([&](int s, uint32_t c, int l, uint32_t gl) {
    const uint32_t q = s_pos[wave][s] + (uint32_t)__popcll(s_mask[wave][s] & ((1ull << l) - 1ull));
    if (q < rows_all) a.rec[q] = make_uint2(gl, c);  // always; a safeguard
  });
}

// The pair stages' blocks of the group are known on the device only (the host
// knows the capacity, some six times the records), so a fixed grid strides over
// them: a workgroup launched for nothing costs 0.4 ns, and there would be tens
// of thousands of them.
constexpr int64_t kPairGrid = 8192;

__device__ __forceinline__ uint32_t group_blocks(const BinArgs& a) {
  return a.blk_base[a.s0 + a.sn] - a.blk_base[a.s0];
}

// The strip of the group (and the first record and record count within it)
// that block b of the pair stages belongs to.
struct RecSpan {
  int strip;
  uint32_t first, count;
};

__device__ __forceinline__ RecSpan rec_span(const BinArgs& a, uint32_t b, int* s_strip) {
  if (threadIdx.x == 0) *s_strip = 0;
  __syncthreads();
  const uint32_t f = a.blk_base[a.s0];
  for (int i = threadIdx.x; i < a.sn; i += kRecThreads)
    if (a.blk_base[a.s0 + i] - f <= b && b < a.blk_base[a.s0 + i + 1] - f) *s_strip = i;
  __syncthreads();
  RecSpan q{*s_strip, 0u, 0u};
  const int s = a.s0 + q.strip;
  const uint32_t seg = b - (a.blk_base[s] - a.blk_base[a.s0]);
  q.first = a.row_base[s] + seg * kRecBlock;
  q.count = min((uint32_t)kRecBlock, a.row_base[s + 1] - q.first);
  return q;
}

// Pairs per column of 512 records: a difference array, then its prefix.
__global__ void __launch_bounds__(kRecThreads) bin_hist_kernel(BinBatch batch) {
  const BinArgs& a = batch.v[blockIdx.z];
  __shared__ int s_diff[kStripCols + 1];
  __shared__ int s_red[kRecThreads / kWave];
  __shared__ int s_strip;
  if (*a.eff_total == 0u) return;
  static_assert(kRecThreads == kStripCols, "a thread per column");
  const int tid = threadIdx.x;
  const uint32_t blocks = group_blocks(a);
  for (uint32_t b = blockIdx.x; b < blocks; b += gridDim.x) {
    const RecSpan q = rec_span(a, b, &s_strip);
    s_diff[tid] = 0;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kRecItems; ++k) {
      const uint32_t i = (uint32_t)(k * kRecThreads + tid);
      if (i < q.count) {
        const uint32_t c = a.rec[q.first + i].y;
        atomicAdd(&s_diff[c & 0xffu], 1);
        atomicAdd(&s_diff[(c >> 8) + 1u], -1);
      }
    }
    __syncthreads();
    const int d = s_diff[tid];
    int tot;
    const int ex = block_exclusive_scan<kRecThreads, int>(d, s_red, &tot);
    if (tid < a.cols) a.hist[(int64_t)b * a.cols + tid] = (uint32_t)(ex + d);
  }
}

// A workgroup per strip of the group, 256 threads over its columns in each of
// four quarters of its blocks: the columns' pairs, the tiles' ranges, and the
// first list position of every (block, column).
__global__ void __launch_bounds__(1024) bin_offsets_kernel(BinBatch batch) {
  const BinArgs& a = batch.v[blockIdx.z];
  if ((int)blockIdx.x >= a.sn) return;  // as in strip_scan_kernel
  __shared__ uint32_t s_part[4][kStripCols];
  __shared__ uint32_t s_red[1024 / kWave];
  const int tid = threadIdx.x, col = tid & (kStripCols - 1), part = tid / kStripCols;
  const int64_t s = (int64_t)a.s0 + blockIdx.x;
  const int64_t ty = s / a.sc;
  const int tx = (int)(s % a.sc) * kStripCols + col;
  const bool in = col < a.cols && tx < a.tiles_x;
  const bool valid = in && (a.bits == nullptr || (a.bits[ty * a.wpr + (tx >> 6)] >> (tx & 63)) & 1ull);
  const bool none = *a.eff_total == 0u;
  const uint32_t b0 = a.blk_base[s] - a.blk_base[a.s0], nb = none ? 0u : a.blk_base[s + 1] - a.blk_base[s];
  const uint32_t per = (nb + 3u) / 4u, f = min(nb, part * per), l = min(nb, f + per);
  uint32_t* h = a.hist + (int64_t)b0 * a.cols + col;
  uint32_t sum = 0;
  if (valid)
#pragma unroll 8
    for (uint32_t b = f; b < l; ++b) sum += h[(int64_t)b * a.cols];
  s_part[part][col] = sum;
  __syncthreads();
  uint32_t tot = 0;
  if (part == 0) tot = s_part[0][col] + s_part[1][col] + s_part[2][col] + s_part[3][col];
  uint32_t all;
  uint32_t run = block_exclusive_scan<1024, uint32_t>(tot, s_red, &all);
  if (part == 0) {
    run += a.pair_base[s];
    if (in) a.ranges[ty * a.tiles_x + tx] = !none && tot > 0 ? make_uint2(run, run + tot) : make_uint2(0u, 0u);
    for (int q = 0; q < 4; ++q) {
      const uint32_t c = s_part[q][col];
      s_part[q][col] = run;
      run += c;
    }
  }
  __syncthreads();
  run = s_part[part][col];
  if (valid)
#pragma unroll 8
    for (uint32_t b = f; b < l; ++b) {
      const uint32_t c = h[(int64_t)b * a.cols];
      h[(int64_t)b * a.cols] = run;
      run += c;
    }
}

// Lists.  A wave takes 64 consecutive records at a time: each sets its bit in
// the masks of its columns, then its rank in a column's list is the mask's
// earlier bits.  The masks and running positions are the wave's own, and a
// wave's LDS operations execute in order, so the rounds need no barrier.  The
// ids go to LDS, column after column, and from there to the lists in runs (512
// records put ~30 ids in each list): written to the lists one by one they were
// 4-byte requests to as many cache lines, which bound the kernel at the L2
// (42M pairs: 229 us, now 141).  A block with more ids than the buffer holds writes them one by
// one.
constexpr int kPlaceIds = 4096;

template <int kCols>
__global__ void __launch_bounds__(kRecThreads) bin_place_kernel(BinBatch batch) {
  const BinArgs& a = batch.v[blockIdx.z];
  constexpr int kWaves = kRecThreads / kWave;
  __shared__ uint64_t s_mask[kWaves][kCols];
  __shared__ uint32_t s_run[kWaves][kCols];
  __shared__ uint32_t s_first[kCols];  // list position of a column's first id, less its place in the buffer
  __shared__ uint32_t s_ids[kPlaceIds];
  __shared__ uint8_t s_col[kPlaceIds];
  __shared__ uint32_t s_red[kWaves];
  __shared__ int s_strip;
  static_assert(kWaves * (kCols + 1) <= kPlaceIds, "the difference arrays fit the id buffer");
  int* const diff = reinterpret_cast<int*>(s_ids);  // [kWaves][kCols + 1], before the ids
  const uint32_t total = *a.eff_total;
  if (total == 0u) return;
  const int tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
  const uint32_t blocks = group_blocks(a);
  for (uint32_t blk = blockIdx.x; blk < blocks; blk += gridDim.x) {
    const RecSpan q = rec_span(a, blk, &s_strip);
    const int64_t s = (int64_t)a.s0 + q.strip;
    const int64_t ty = s / a.sc;
    const int x0 = (int)(s % a.sc) * kStripCols;
    const uint64_t* brow = a.bits != nullptr ? a.bits + ty * a.wpr + (x0 >> 6) : nullptr;
    auto listed = [&](int x) { return brow == nullptr || (brow[x >> 6] >> (x & 63)) & 1ull; };
    for (int i = tid; i < kWaves * kCols; i += kRecThreads) (&s_mask[0][0])[i] = 0ull;
    for (int i = tid; i < kWaves * (kCols + 1); i += kRecThreads) diff[i] = 0;
    __syncthreads();
    // each wave takes 64 kRecItems consecutive records
    uint2 rec[kRecItems];
#pragma unroll
    for (int k = 0; k < kRecItems; ++k) {
      const uint32_t i = (uint32_t)((wave * kRecItems + k) * kWave + lane);
      rec[k] = i < q.count ? a.rec[q.first + i] : make_uint2(0u, 0xffu);  // past the end: an empty interval
      if (i < q.count) {
        atomicAdd(&diff[wave * (kCols + 1) + (int)(rec[k].y & 0xffu)], 1);
        atomicAdd(&diff[wave * (kCols + 1) + (int)(rec[k].y >> 8) + 1], -1);
      }
    }
    __syncthreads();
    {
      // the wave's ids per column
      constexpr int kPer = kCols / kWave;
      int d[kPer], sum = 0;
#pragma unroll
      for (int k = 0; k < kPer; ++k) {
        d[k] = diff[wave * (kCols + 1) + lane * kPer + k];
        sum += d[k];
      }
      int run = wave_inclusive_scan_i_dpp(sum) - sum;
#pragma unroll
      for (int k = 0; k < kPer; ++k) {
        run += d[k];
        s_run[wave][lane * kPer + k] = (uint32_t)run;
      }
    }
    __syncthreads();
    uint32_t ids = 0;
    if (tid < a.cols && listed(tid))
      for (int w = 0; w < kWaves; ++w) ids += s_run[w][tid];
    uint32_t block_ids;
    uint32_t run = block_exclusive_scan<kRecThreads, uint32_t>(ids, s_red, &block_ids);
    if (tid < a.cols) {
      s_first[tid] = a.hist[(int64_t)blk * a.cols + tid] - run;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        const uint32_t c = s_run[w][tid];
        s_run[w][tid] = run;
        run += c;
      }
    }
    __syncthreads();
    const bool buffered = block_ids <= (uint32_t)kPlaceIds;  // workgroup-uniform
    auto put = [&](uint32_t pos, int x, uint32_t id) {
      if (pos >= total) return;  // never; a safeguard
      a.vals[pos] = id;
      if (a.keys64 != nullptr)
        a.keys64[pos] = ((uint64_t)(ty * a.tiles_x + x0 + x) << 32) | (uint64_t)__float_as_uint(a.depth[id]);
    };
    const uint64_t below = lanes_below();
    uint64_t* const mask = s_mask[wave];
    uint32_t* const base = s_run[wave];
#pragma unroll
    for (int k = 0; k < kRecItems; ++k) {
      const int xl = (int)(rec[k].y & 0xffu), xh = (int)(rec[k].y >> 8);
      for (int x = xl; x <= xh; ++x)
        __hip_atomic_fetch_or(&mask[x], 1ull << lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      for (int x = xl; x <= xh; ++x) {
        if (!listed(x)) continue;
        const uint32_t lp = base[x] + (uint32_t)__popcll(mask[x] & below);
        if (!buffered) {
          put(s_first[x] + lp, x, rec[k].x);
        } else if (lp < (uint32_t)kPlaceIds) {  // always (the counts are the masks'); a safeguard
          s_ids[lp] = rec[k].x;
          s_col[lp] = (uint8_t)x;
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      for (int x = lane; x < kCols; x += kWave) {
        const uint64_t m = mask[x];
        if (m != 0ull) {
          base[x] += (uint32_t)__popcll(m);
          mask[x] = 0ull;
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    if (buffered)
      for (uint32_t i = tid; i < block_ids; i += kRecThreads) put(s_first[s_col[i]] + i, s_col[i], s_ids[i]);
    __syncthreads();  // before the next block clears the masks and the difference arrays
  }
}

// ------------------------------------------------------------------ workspace
struct SortWs {
  unsigned long long* counts;   // [2] pairs (blocking call's readback)
  uint32_t* eff_total;          // all pairs when they fit the capacity, else 0
  uint32_t* n_keyed;            // Gaussians with a non-empty rectangle
  uint32_t* dhist;              // [256][hstride] per-block digit counts of the depth pass being run
  uint32_t* dhoffs;             // [256][hstride] their prefix per digit
  uint32_t* ddtot;              // [256] digit totals
  int hstride;
  uint32_t* dkeys[2];           // [n] depth keys (ping-pong)
  uint32_t* dvals[2];           // [n] ids
  uint32_t* ids_sorted;         // [n] Gaussians in depth order
  uint32_t* part;               // few Gaussians: [chunks][n] partial ranks
  int4* rects;                  // [n] clamped rectangles (kept by a depth-prefix call)
  uint16_t* spans;              // [kb][span_rows]
  int2* rowinfo;                // [n]
  int64_t kb;                   // blocks of depth positions
  int span_rows, group;         // rows of a block whose intervals are kept; strips in a group
  uint32_t* rows_tab;           // [group][kb]
  uint32_t* pairs_tab;
  unsigned long long* row_tot;  // [n_tiles] (at most a strip per tile)
  unsigned long long* pair_tot;
  uint32_t* row_base;           // [n_tiles + 1]
  uint32_t* pair_base;
  uint32_t* blk_base;
  uint64_t* bits;               // [at most n_tiles] words
  uint2* rec;                   // [capacity]
  uint32_t* hist;               // [capacity / kRecBlock + group][kStripCols or fewer]
  size_t bytes;
};

// The workspace holds the tables of any grid of up to kTilesAlways tiles (36
// bytes each), so a caller need not give the grid's size: the calls of one
// workspace may have several grids.
constexpr int64_t kTilesAlways = 1 << 16, kTilesUnknown = 1 << 20;

static SortWs layout(void* ws, int64_t n, int64_t capacity, int64_t n_tiles) {
  const int64_t cap = std::max<int64_t>(capacity, 1), nn = std::max<int64_t>(n, 1);
  const int64_t nt = std::max(n_tiles, kTilesAlways);
  size_t o = 0;
  char* b = (char*)ws;
  auto take = [&](size_t bytes) {
    char* p = b ? b + o : nullptr;
    o += align_up(bytes, 256);
    return (void*)p;
  };
  SortWs w;
  w.counts = (unsigned long long*)take(4 * sizeof(unsigned long long));
  w.eff_total = (uint32_t*)(w.counts ? w.counts + 2 : nullptr);
  w.n_keyed = (uint32_t*)(w.counts ? w.counts + 3 : nullptr);
  w.hstride = (int)(ceil_div(ceil_div(nn, kDepthBlockKeys), 4) * 4);
  w.dhist = (uint32_t*)take(sizeof(uint32_t) * kDepthDigits * w.hstride);
  w.dhoffs = (uint32_t*)take(sizeof(uint32_t) * kDepthDigits * w.hstride);
  w.ddtot = (uint32_t*)take(sizeof(uint32_t) * kDepthDigits);
  for (int k = 0; k < 2; ++k) {
    w.dkeys[k] = (uint32_t*)take(sizeof(uint32_t) * nn);
    w.dvals[k] = (uint32_t*)take(sizeof(uint32_t) * nn);
  }
  w.ids_sorted = w.dvals[0];  // the last pass's target
  w.part = (uint32_t*)take(nn <= kSmallSort ? sizeof(uint32_t) * nn * ceil_div(nn, kRankChunk) : 0);
  w.rects = (int4*)take(sizeof(int4) * nn);
  w.kb = ceil_div(nn, kRowThreads);
  const bool few = nn <= kFewGaussians;
  const int64_t group = few ? kGroupFew : kGroup;
  w.span_rows = few ? kSpansFew : kSpans;
  w.group = (int)group;
  w.spans = (uint16_t*)take(sizeof(uint16_t) * w.span_rows * w.kb);
  w.rowinfo = (int2*)take(sizeof(int2) * nn);
  w.rows_tab = (uint32_t*)take(sizeof(uint32_t) * group * w.kb);
  w.pairs_tab = (uint32_t*)take(sizeof(uint32_t) * group * w.kb);
  w.row_tot = (unsigned long long*)take(sizeof(unsigned long long) * nt);
  w.pair_tot = (unsigned long long*)take(sizeof(unsigned long long) * nt);
  w.row_base = (uint32_t*)take(sizeof(uint32_t) * (nt + 1));
  w.pair_base = (uint32_t*)take(sizeof(uint32_t) * (nt + 1));
  w.blk_base = (uint32_t*)take(sizeof(uint32_t) * (nt + 1));
  w.bits = (uint64_t*)take(sizeof(uint64_t) * nt);
  w.rec = (uint2*)take(sizeof(uint2) * cap);
  w.hist = (uint32_t*)take(sizeof(uint32_t) * (cap / kRecBlock + group + 1) * kStripCols);
  w.bytes = o;
  return w;
}

// The depth orders of the views' Gaussians with a non-empty rectangle.
static void sort_depth(const DepthBatch& d, int views, int64_t n, hipStream_t s) {
  const unsigned nv = (unsigned)views;
  if (n <= kSmallSort) {
    const int chunks = (int)ceil_div(n, kRankChunk);
    const unsigned blocks = (unsigned)ceil_div(n, kRankThreads);
    hipLaunchKernelGGL(rank_kernel, dim3(blocks, (unsigned)chunks, nv), dim3(kRankThreads), 0, s, d);
    hipLaunchKernelGGL(rank_place_kernel, dim3(blocks, 1, nv), dim3(kRankThreads), 0, s, d, chunks);
    return;
  }
  const dim3 grid((unsigned)ceil_div(n, kDepthBlockKeys), 1, nv), block(kSortThreads);
  hipLaunchKernelGGL(key_kernel, grid, block, 0, s, d);
  for (int p = 0; p < 4; ++p) {  // the ids end in vals[0]
    if (p > 0) hipLaunchKernelGGL(depth_hist_kernel, grid, block, 0, s, d, p);
    hipLaunchKernelGGL(digit_scan_kernel, dim3(kDepthDigits, 1, nv), dim3(1024), 0, s, d, p);
    if (p == 0)
      hipLaunchKernelGGL((depth_pass_kernel<true, false>), grid, block, 0, s, d, p);
    else if (p < 3)
      hipLaunchKernelGGL((depth_pass_kernel<false, false>), grid, block, 0, s, d, p);
    else
      hipLaunchKernelGGL((depth_pass_kernel<false, true>), grid, block, 0, s, d, p);
  }
}

static int64_t strips_of(const BinArgs& a) { return (int64_t)a.sc * a.tiles_y; }

// The lists of the depth positions that each view's arguments describe
// (pos0 .. pos_end).
template <bool kWide>
static void list_pairs(BinBatch& b, int views, hipStream_t s) {
  const int64_t group_strips = b.v[0].group;  // of the Gaussian count: the same in all views
  const size_t span_bytes = kWide ? 0 : sizeof(uint16_t) * b.v[0].span_rows;
  const unsigned nv = (unsigned)views;
  int64_t strips = 0, positions = 0, capacity = 0;
  int rows = 0, cols = 0;
  bool subset = false;
  for (int k = 0; k < views; ++k) {
    strips = std::max(strips, strips_of(b.v[k]));
    positions = std::max(positions, b.v[k].pos_end - b.v[k].pos0);
    capacity = std::max(capacity, b.v[k].capacity);
    rows = std::max(rows, b.v[k].tiles_y);
    cols = std::max(cols, b.v[k].cols);
    subset = subset || b.v[k].tile_slot != nullptr;
  }
  const unsigned kb = (unsigned)ceil_div(positions, kRowThreads);
  unsigned sn = 0;
  auto group = [&](int64_t s0) {
    sn = 0;
    for (int k = 0; k < views; ++k) {
      BinArgs& a = b.v[k];
      a.s0 = (int)s0;
      a.sn = (int)std::min<int64_t>(group_strips, strips_of(a) - s0);
      a.y0 = (int)(s0 / a.sc);
      a.y1 = (int)((s0 + a.sn - 1) / a.sc) + 1;
      sn = std::max(sn, (unsigned)a.sn);
    }
  };
  auto count = [&] {
    if (kb > 0)
      hipLaunchKernelGGL(bin_count_kernel<kWide>, dim3(kb, 1, nv), dim3(kRowThreads),
                         2 * sizeof(uint32_t) * sn + span_bytes, s, b);
    hipLaunchKernelGGL(strip_scan_kernel, dim3(sn, 1, nv), dim3(1024), 0, s, b);
  };
  if (subset && !b.v[0].counted)
    hipLaunchKernelGGL(tile_bits_kernel, dim3((unsigned)rows, 1, nv), dim3(kWave), 0, s, b);
  const bool counted = b.v[0].counted;  // a view's lists resumed, alone in its batch
  for (int64_t s0 = 0; s0 < strips && !counted; s0 += group_strips) {
    group(s0);
    count();
  }
  hipLaunchKernelGGL(strip_base_kernel, dim3(1, 1, nv), dim3(1024), 0, s, b);
  for (int64_t s0 = 0; s0 < strips; s0 += group_strips) {
    group(s0);
    if (strips > group_strips) count();  // the tables hold one group
    if (kb > 0 && capacity > 0) {
      const unsigned nb = (unsigned)std::min<int64_t>(capacity / kRecBlock + sn, kPairGrid);
      hipLaunchKernelGGL(bin_rows_kernel<kWide>, dim3(kb, (unsigned)ceil_div((int)sn, kSub), nv),
                         dim3(kRowThreads), span_bytes, s, b);
      hipLaunchKernelGGL(bin_hist_kernel, dim3(nb, 1, nv), dim3(kRecThreads), 0, s, b);
      hipLaunchKernelGGL(bin_offsets_kernel, dim3(sn, 1, nv), dim3(1024), 0, s, b);
      if (cols <= kStripCols / 2)  // half the LDS: more workgroups per compute unit
        hipLaunchKernelGGL(bin_place_kernel<kStripCols / 2>, dim3(nb, 1, nv), dim3(kRecThreads), 0, s, b);
      else
        hipLaunchKernelGGL(bin_place_kernel<kStripCols>, dim3(nb, 1, nv), dim3(kRecThreads), 0, s, b);
    } else {
      hipLaunchKernelGGL(bin_offsets_kernel, dim3(sn, 1, nv), dim3(1024), 0, s, b);
    }
  }
}

// Views of more strips than one group, or of strips cut by columns, go one by
// one; the others together.
static void list_all(BinBatch& b, int views, hipStream_t s) {
  bool together = true;
  for (int k = 0; k < views; ++k) together = together && b.v[k].sc == 1 && strips_of(b.v[k]) <= b.v[k].group;
  if (together) {
    list_pairs<false>(b, views, s);
    return;
  }
  for (int k = 0; k < views; ++k) {
    BinBatch one{};
    one.v[0] = b.v[k];
    if (one.v[0].sc > 1) list_pairs<true>(one, 1, s);
    else list_pairs<false>(one, 1, s);
  }
}

// What both calls share of BinArgs; tile_slot nullable.
static BinArgs bin_args(const SortWs& w, const float* splat, const int32_t* tile_slot, int tiles_x, int tiles_y,
                        float alpha_min, uint32_t* vals, uint32_t* ranges, int64_t capacity,
                        unsigned long long* out) {
  BinArgs a{};
  a.splat = (const float4*)splat;
  a.tiles_x = tiles_x;
  a.tiles_y = tiles_y;
  a.wpr = (int)ceil_div(tiles_x, kWave);
  a.sc = (int)ceil_div(tiles_x, kStripCols);
  a.cols = std::min(tiles_x, kStripCols);
  // 2 ln(1/alpha_min) with a 0.1 % margin, rounded up to a multiple of 1/64
  a.lia = std::log(1.0 / (double)alpha_min);
  a.tau = std::ceil(128.0 * a.lia * 1.001) / 64.0;
  a.kb = w.kb;
  a.span_rows = w.span_rows;
  a.group = w.group;
  a.rows_tab = w.rows_tab;
  a.pairs_tab = w.pairs_tab;
  a.spans = w.spans;
  a.rowinfo = w.rowinfo;
  a.row_tot = w.row_tot;
  a.pair_tot = w.pair_tot;
  a.row_base = w.row_base;
  a.pair_base = w.pair_base;
  a.blk_base = w.blk_base;
  a.eff_total = w.eff_total;
  a.rec = w.rec;
  a.hist = w.hist;
  a.vals = vals;
  a.ranges = (uint2*)ranges;
  a.tile_slot = tile_slot;
  a.bits = tile_slot != nullptr ? w.bits : nullptr;
  a.m = -1;
  a.capacity = capacity;
  a.counts = w.counts;
  a.out = out;
  return a;
}

}  // namespace tgs

using namespace tgs;

extern "C" size_t tgs_bin_sort_workspace_size(int64_t n, int64_t capacity, int32_t n_tiles) {
  if (n < 0 || capacity < 0) return 0;
  return layout(nullptr, n, capacity, n_tiles > 0 ? n_tiles : kTilesUnknown).bytes;
}

// One view's call, after its argument checks: what goes into the batches.
// prefix >= 0: the lists hold the pairs of the first `prefix` Gaussians in
// (depth, id) order only (every Gaussian when prefix >= n) and out[2] is the
// prefix call's estimate; -1: whole lists.  out nullable.
static void bin_sort_view(DepthArgs& d, BinArgs& a, const int32_t* rect, const float* splat, const float* depth,
                          int64_t n, const int32_t* tile_slot, int32_t tiles_x, int32_t tiles_y, float alpha_min,
                          uint64_t* keys, uint32_t* vals, int64_t capacity, uint32_t* ranges, uint8_t* touched,
                          const SortWs& w, unsigned long long* out, int64_t prefix) {
  d.rect = (const int4*)rect;
  d.depth = depth;
  d.n = (uint32_t)n;
  d.tiles_x = tiles_x;
  d.tiles_y = tiles_y;
  d.stride = w.hstride;
  for (int k = 0; k < 2; ++k) {
    d.keys[k] = w.dkeys[k];
    d.vals[k] = w.dvals[k];
  }
  d.hist = w.dhist;
  d.hoffs = w.dhoffs;
  d.dtot = w.ddtot;
  d.n_keyed = w.n_keyed;
  d.rects = prefix >= 0 ? w.rects : nullptr;
  d.part = w.part;
  a = bin_args(w, splat, tile_slot, tiles_x, tiles_y, alpha_min, vals, ranges, capacity, out);
  a.n_keyed = w.n_keyed;
  a.pos0 = 0;
  a.pos_end = prefix >= 0 ? std::min(prefix, n) : n;
  a.m = prefix >= 0 ? a.pos_end : -1;
  a.ids = w.ids_sorted;
  a.rect = (const int4*)rect;
  a.touched = touched;
  a.keys64 = keys;
  a.depth = depth;
}

// Queued on the stream, no host wait.
static int32_t bin_sort_queue(const DepthBatch& d, BinBatch& b, int views, int64_t n, hipStream_t s,
                              const char* who) {
  if (n > 0)
    sort_depth(d, views, n, s);
  else
    for (int k = 0; k < views; ++k)
      hipLaunchKernelGGL(set_kernel<uint32_t>, dim3(1), dim3(64), 0, s, d.v[k].n_keyed, 0u);
  list_all(b, views, s);
  return hip_status(who);
}

static int32_t bin_sort_one(const int32_t* rect, const float* splat, const float* depth, int64_t n,
                            const int32_t* tile_slot, int32_t tiles_x, int32_t tiles_y, float alpha_min,
                            uint64_t* keys, uint32_t* vals, int64_t capacity, uint32_t* ranges, uint8_t* touched,
                            const SortWs& w, hipStream_t s, const char* who, unsigned long long* out,
                            int64_t prefix = -1) {
  DepthBatch d{};
  BinBatch b{};
  bin_sort_view(d.v[0], b.v[0], rect, splat, depth, n, tile_slot, tiles_x, tiles_y, alpha_min, keys, vals, capacity,
                ranges, touched, w, out, prefix);
  return bin_sort_queue(d, b, 1, n, s, who);
}

// A call that did not fit its capacity, taken up again with larger arrays: the
// depth order, the tile bits and the counts are in its workspace w1 (whose
// layout holds the arrays that grow with the capacity last), so the records
// and lists are all that is left: an autograd pass over 300k Gaussians, whose
// first capacity is too small, 658 us with the whole call repeated, 550 so.
static void resume_view(BinArgs& a, const SortWs& w1) {
  a.counted = true;
  a.ids = w1.ids_sorted;
  a.n_keyed = w1.n_keyed;
  a.bits = a.tile_slot != nullptr ? w1.bits : nullptr;
  a.rows_tab = w1.rows_tab;
  a.pairs_tab = w1.pairs_tab;
  a.spans = w1.spans;
  a.rowinfo = w1.rowinfo;
  a.row_tot = w1.row_tot;
  a.pair_tot = w1.pair_tot;
  a.row_base = w1.row_base;
  a.pair_base = w1.pair_base;
  a.blk_base = w1.blk_base;
}

// The continuation of depth-prefix lists: the pairs of the Gaussians from
// depth rank `prefix` on in the flagged tiles, from the depth order and the
// rectangles that the prefix call left in its workspace w1, with the tables
// and buffers of w2.
static BinArgs continue_view(const float* splat, int64_t n, const int32_t* flag_slot, const uint32_t* n_flagged,
                             int32_t tiles_x, int32_t tiles_y, float alpha_min, int64_t prefix, uint32_t* vals2,
                             int64_t capacity2, uint32_t* ranges2, const SortWs& w1, const SortWs& w2,
                             unsigned long long* out) {
  BinArgs a = bin_args(w2, splat, flag_slot, tiles_x, tiles_y, alpha_min, vals2, ranges2, capacity2, out);
  a.n_keyed = w1.n_keyed;
  a.pos0 = std::min(prefix, n);
  a.pos_end = n;
  a.ids = w1.ids_sorted;
  a.rect = w1.rects;
  a.n_flagged = n_flagged;
  return a;
}

static int32_t bin_sort_check(const int32_t* rect, const float* splat, const float* depth, int64_t n,
                              int32_t tiles_x, int32_t tiles_y, float alpha_min, uint32_t* vals, int64_t capacity,
                              uint32_t* ranges, void* ws, size_t ws_bytes, const SortWs& w, const char* who) {
  TGS_REQUIRE(n >= 0 && n < (1ll << 31), "%s: n out of range", who);
  TGS_REQUIRE(tiles_x > 0 && tiles_y > 0 && (int64_t)tiles_x * tiles_y < (1ll << 30), "%s: bad tile grid", who);
  TGS_REQUIRE(capacity >= 0 && capacity < (1ll << 32), "%s: capacity out of range", who);
  TGS_REQUIRE(alpha_min > 0.f && alpha_min < 1.f, "%s: alpha_min %g not in (0, 1)", who, (double)alpha_min);
  TGS_REQUIRE(vals && ranges && ws, "%s: null pointer", who);  // keys may be null
  TGS_REQUIRE(n == 0 || (rect && splat && depth), "%s: null rect/splat/depth", who);
  TGS_REQUIRE(((uintptr_t)rect & 15) == 0 && ((uintptr_t)splat & 15) == 0 && ((uintptr_t)ws & 15) == 0,
              "%s: rect, splat and ws must be 16-byte aligned", who);
  TGS_REQUIRE(ws_bytes >= w.bytes, "%s: workspace %zu bytes < %zu", who, ws_bytes, w.bytes);
  return TGS_OK;
}

// Tiles of a grid for the layout; 0 for a grid that the checks refuse.
static int64_t grid_tiles(int32_t tiles_x, int32_t tiles_y) {
  return tiles_x > 0 && tiles_y > 0 ? (int64_t)tiles_x * tiles_y : 0;
}

extern "C" int32_t tgs_bin_sort_async(const int32_t* rect, const float* splat, const float* depth, int64_t n,
                                      const int32_t* tile_slot, int32_t tiles_x, int32_t tiles_y, float alpha_min,
                                      uint64_t* keys, uint32_t* vals, int64_t capacity, uint32_t* ranges,
                                      uint8_t* touched, int64_t* counts, void* ws, size_t ws_bytes, void* stream) {
  const SortWs w = layout(ws, n, capacity, grid_tiles(tiles_x, tiles_y));
  if (int32_t e = bin_sort_check(rect, splat, depth, n, tiles_x, tiles_y, alpha_min, vals, capacity, ranges, ws,
                                 ws_bytes, w, "tgs_bin_sort_async"))
    return e;
  TGS_REQUIRE(counts != nullptr && ((uintptr_t)counts & 7) == 0,
              "tgs_bin_sort_async: counts must be an 8-byte aligned device pointer");
  return bin_sort_one(rect, splat, depth, n, tile_slot, tiles_x, tiles_y, alpha_min, keys, vals, capacity, ranges,
                      touched, w, as_stream(stream), "tgs_bin_sort_async", (unsigned long long*)counts);
}

extern "C" int32_t tgs_bin_sort_resume_async(const int32_t* rect, const float* splat, const float* depth, int64_t n,
                                             const int32_t* tile_slot, int32_t tiles_x, int32_t tiles_y,
                                             float alpha_min, const void* ws1, size_t ws1_bytes, int64_t capacity1,
                                             uint64_t* keys, uint32_t* vals, int64_t capacity, uint32_t* ranges,
                                             uint8_t* touched, int64_t* counts, void* ws, size_t ws_bytes,
                                             void* stream) {
  const char* who = "tgs_bin_sort_resume_async";
  const int64_t n_t = grid_tiles(tiles_x, tiles_y);
  const SortWs w = layout(ws, n, capacity, n_t);
  if (int32_t e = bin_sort_check(rect, splat, depth, n, tiles_x, tiles_y, alpha_min, vals, capacity, ranges, ws,
                                 ws_bytes, w, who))
    return e;
  TGS_REQUIRE(counts != nullptr && ((uintptr_t)counts & 7) == 0, "%s: counts must be an 8-byte aligned device pointer",
              who);
  TGS_REQUIRE(ws1 != nullptr && ((uintptr_t)ws1 & 15) == 0 && ws1 != ws && capacity1 >= 0 && capacity1 < (1ll << 32),
              "%s: bad first workspace", who);
  const SortWs w1 = layout((void*)ws1, n, capacity1, n_t);
  TGS_REQUIRE(ws1_bytes >= w1.bytes, "%s: first workspace %zu bytes < %zu", who, ws1_bytes, w1.bytes);
  DepthBatch d{};
  BinBatch b{};
  bin_sort_view(d.v[0], b.v[0], rect, splat, depth, n, tile_slot, tiles_x, tiles_y, alpha_min, keys, vals, capacity,
                ranges, touched, w, (unsigned long long*)counts, -1);
  resume_view(b.v[0], w1);
  // more strips than one group: their tables were overwritten group by group
  if (b.v[0].sc > 1 || strips_of(b.v[0]) > b.v[0].group) b.v[0].counted = false;
  list_all(b, 1, as_stream(stream));
  return hip_status(who);
}

extern "C" int32_t tgs_bin_sort_prefix_async(const int32_t* rect, const float* splat, const float* depth, int64_t n,
                                             const int32_t* tile_slot, int32_t tiles_x, int32_t tiles_y,
                                             float alpha_min, int64_t prefix, uint64_t* keys, uint32_t* vals,
                                             int64_t capacity, uint32_t* ranges, uint8_t* touched, int64_t* counts,
                                             void* ws, size_t ws_bytes, void* stream) {
  const SortWs w = layout(ws, n, capacity, grid_tiles(tiles_x, tiles_y));
  if (int32_t e = bin_sort_check(rect, splat, depth, n, tiles_x, tiles_y, alpha_min, vals, capacity, ranges, ws,
                                 ws_bytes, w, "tgs_bin_sort_prefix_async"))
    return e;
  TGS_REQUIRE(prefix >= 0, "tgs_bin_sort_prefix_async: negative prefix");
  TGS_REQUIRE(counts != nullptr && ((uintptr_t)counts & 7) == 0,
              "tgs_bin_sort_prefix_async: counts must be an 8-byte aligned device pointer");
  return bin_sort_one(rect, splat, depth, n, tile_slot, tiles_x, tiles_y, alpha_min, keys, vals, capacity, ranges,
                      touched, w, as_stream(stream), "tgs_bin_sort_prefix_async", (unsigned long long*)counts, prefix);
}

// The views in batches, each kernel launched once for up to kBatch of them.
extern "C" int32_t tgs_bin_sort_views_async(const tgs_bin_view* views, int32_t n_views, int64_t n, float alpha_min,
                                            int64_t prefix, void* stream) {
  const char* who = "tgs_bin_sort_views_async";
  TGS_REQUIRE(n_views >= 0 && (n_views == 0 || views != nullptr), "%s: bad view list", who);
  TGS_REQUIRE(prefix >= -1, "%s: prefix below -1", who);
  for (int k = 0; k < n_views; ++k) {
    const tgs_bin_view& v = views[k];
    const SortWs w = layout(v.ws, n, v.capacity, grid_tiles(v.tiles_x, v.tiles_y));
    if (int32_t e = bin_sort_check(v.rect, v.splat, v.depth, n, v.tiles_x, v.tiles_y, alpha_min, v.vals, v.capacity,
                                   v.ranges, v.ws, v.ws_bytes, w, who))
      return e;
    TGS_REQUIRE(v.counts != nullptr && ((uintptr_t)v.counts & 7) == 0,
                "%s: counts must be an 8-byte aligned device pointer", who);
  }
  for (int k0 = 0; k0 < n_views; k0 += kBatch) {
    const int nv = std::min(kBatch, n_views - k0);
    DepthBatch d{};
    BinBatch b{};
    for (int k = 0; k < nv; ++k) {
      const tgs_bin_view& v = views[k0 + k];
      bin_sort_view(d.v[k], b.v[k], v.rect, v.splat, v.depth, n, v.tile_slot, v.tiles_x, v.tiles_y, alpha_min, v.keys,
                    v.vals, v.capacity, v.ranges, v.touched,
                    layout(v.ws, n, v.capacity, grid_tiles(v.tiles_x, v.tiles_y)), (unsigned long long*)v.counts,
                    prefix);
    }
    if (int32_t e = bin_sort_queue(d, b, nv, n, as_stream(stream), who)) return e;
  }
  return TGS_OK;
}

extern "C" int32_t tgs_bin_sort_continue_async(const float* splat, int64_t n, const int32_t* flag_slot,
                                               const uint32_t* n_flagged, int32_t tiles_x, int32_t tiles_y,
                                               float alpha_min, int64_t prefix,
                                               int64_t capacity, const void* ws, size_t ws_bytes, uint32_t* vals2,
                                               int64_t capacity2, uint32_t* ranges2, int64_t* counts2, void* ws2,
                                               size_t ws2_bytes, void* stream) {
  const char* who = "tgs_bin_sort_continue_async";
  TGS_REQUIRE(n >= 0 && n < (1ll << 31) && prefix >= 0, "%s: n or prefix out of range", who);
  TGS_REQUIRE(tiles_x > 0 && tiles_y > 0 && (int64_t)tiles_x * tiles_y < (1ll << 30), "%s: bad tile grid", who);
  TGS_REQUIRE(capacity >= 0 && capacity2 >= 0 && capacity2 < (1ll << 32), "%s: capacity out of range", who);
  TGS_REQUIRE(alpha_min > 0.f && alpha_min < 1.f, "%s: alpha_min %g not in (0, 1)", who, (double)alpha_min);
  TGS_REQUIRE(splat && flag_slot && ws && vals2 && ranges2 && counts2 && ws2, "%s: null pointer", who);
  TGS_REQUIRE(((uintptr_t)splat & 15) == 0 && ((uintptr_t)ws & 15) == 0 && ((uintptr_t)ws2 & 15) == 0 &&
                  ((uintptr_t)counts2 & 7) == 0,
              "%s: splat, ws and ws2 must be 16-byte, counts2 8-byte aligned", who);
  const int64_t n_t = grid_tiles(tiles_x, tiles_y);
  const SortWs w1 = layout((void*)ws, n, capacity, n_t);
  const SortWs w2 = layout(ws2, n, capacity2, n_t);
  TGS_REQUIRE(ws_bytes >= w1.bytes && ws2_bytes >= w2.bytes, "%s: workspace too small", who);
  BinBatch b{};
  b.v[0] = continue_view(splat, n, flag_slot, n_flagged, tiles_x, tiles_y, alpha_min, prefix, vals2, capacity2, ranges2,
                         w1, w2, (unsigned long long*)counts2);
  list_all(b, 1, as_stream(stream));
  return hip_status(who);
}

extern "C" int32_t tgs_bin_sort(const int32_t* rect, const float* splat, const float* depth, int64_t n,
                                const int32_t* tile_slot, int32_t tiles_x, int32_t tiles_y, float alpha_min,
                                uint64_t* keys, uint32_t* vals, int64_t capacity, uint32_t* ranges,
                                uint8_t* touched, int64_t* n_pairs, void* ws, size_t ws_bytes,
                                void* stream) {
  const SortWs w = layout(ws, n, capacity, grid_tiles(tiles_x, tiles_y));
  if (int32_t e = bin_sort_check(rect, splat, depth, n, tiles_x, tiles_y, alpha_min, vals, capacity, ranges, ws,
                                 ws_bytes, w, "tgs_bin_sort"))
    return e;
  TGS_REQUIRE(n_pairs != nullptr, "tgs_bin_sort: null n_pairs");
  hipStream_t s = as_stream(stream);
  if (int32_t e = bin_sort_one(rect, splat, depth, n, tile_slot, tiles_x, tiles_y, alpha_min, keys, vals, capacity,
                               ranges, touched, w, s, "tgs_bin_sort", nullptr))
    return e;
  // the one synchronisation: the two counts, read back when the stream has run the call
  unsigned long long host[2] = {0, 0};
  if (hipMemcpyAsync(host, w.counts, sizeof(host), hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess)
    return hip_status("tgs_bin_sort: count readback");
  if ((int64_t)host[1] > capacity) {
    *n_pairs = (int64_t)host[1];
    set_error("tgs_bin_sort: %llu pairs exceed capacity %lld", host[1], (long long)capacity);
    return TGS_ERR_CAPACITY;
  }
  *n_pairs = (int64_t)host[0];
  return hip_status("tgs_bin_sort");
}
