// Front-to-back compositing of the sampled pixels (forward) and its adjoint.
//
// One workgroup per sampled tile; a lane owns one sampled pixel of the tile
// (sparse mode: the tile's explicit sample list from the prefix offsets;
// dense mode: all 256 pixels).  The tile's depth-sorted Gaussian range is
// walked in batches of one Gaussian per thread, staged into LDS as a
// tile-local centre, the conic, the opacity and the colour, so every lane
// evaluates the batch from LDS broadcasts.  The walk stops when every lane's
// transmittance has terminated (workgroup vote per batch, wave exit inside).
//
// The backward replays the same walk front to back, recomputing T and the
// accumulated colour from the forward outputs (final colour and the number
// of contributors), so nothing per Gaussian or per (pixel, Gaussian) is
// stored.  Optionally the forward records each pixel's (T, accumulated
// colour) at the first position of every chunk of the list (chunk_begin); the
// backward then runs one workgroup per (tile, chunk) that starts from the
// recorded state.  The replay performs the same operations in the same
// order, so its decisions and transmittances are the unchunked ones (the colour
// behind a Gaussian is formed anew from the recorded state); at 64 samples
// per tile this turns one wave per tile into several, which the SIMDs need
// to hide latency.  The nine screen-space gradients of a Gaussian are moments
// over the pixels, summed by lanes that hold one Gaussian and four pixels, the
// colours' on the matrix cores (see render_bwd_view); the batch's sums then
// leave in one pass of atomics.
//
// The forward and the density walk keep the next batch's records and the ids of
// the one after it in flight while the current batch is evaluated: at 64
// samples per tile a tile is one wave, so there are few waves per SIMD to hide
// memory latency otherwise.  The backward keeps the next ids only (its walk
// needs the registers).
#include <algorithm>

#include "common.h"

namespace tgs {

struct RasterArgs {
  const float4* splat;
  const uint32_t* vals;
  const uint2* ranges;
  // optional second segment of every tile's list (depth-prefix lists and
  // their continuation): the tile's list is vals[ranges[t]] followed by
  // vals2[ranges2[t]]
  const uint32_t* vals2;
  const uint2* ranges2;
  const int32_t* valid_tiles;
  const int32_t* tile_off;
  const uint8_t* pix;
  int tiles_x, tiles_y, width, height;
  float alpha_min, alpha_max, T_min;
  float bg0, bg1, bg2;
  // forward only: 0 plain; 1 depth-prefix pass (marks the tiles with a
  // pixel that ran off its list without the T_min stop, counts the other
  // pixels); 2 continuation pass over the slots cont_list[0 .. *cont_count)
  // (counts only the pixels the prefix pass left open)
  int mode;
  int32_t* cont_slot;     // [n_tiles] -1, or the slot of a marked tile (mode 1)
  uint32_t* cont_list;    // marked slots (written in mode 1, read in mode 2)
  uint32_t* cont_count;   // their number
};

// One tile's list: n1 entries from vals at b1, then len - n1 from vals2 at
// b2.  Positions are list-relative (0 .. len).
struct TileList {
  uint32_t b1, n1, b2, len;
};

__device__ __forceinline__ TileList tile_list(const RasterArgs& a, int tile) {
  const uint2 r = a.ranges[tile];
  TileList L{r.x, r.y - r.x, 0u, r.y - r.x};
  if (a.ranges2 != nullptr) {
    const uint2 q = a.ranges2[tile];
    L.b2 = q.x;
    L.len += q.y - q.x;
  }
  return L;
}

__device__ __forceinline__ uint32_t list_id(const RasterArgs& a, const TileList& L, uint32_t pos) {
  return pos < L.n1 ? a.vals[L.b1 + pos] : a.vals2[L.b2 + (pos - L.n1)];
}

// The alpha decisions must come out bit-identical in the forward and the
// replay, so both evaluate alpha through these functions, written with
// explicit fused operations and no contraction left to the compiler.
//
// The splat record holds the conic Q = [[a, b], [b, c]] in its LDL^T form
// (a, beta = b/a, delta = det Q / a), so that
// d^T Q d = a (dx + beta dy)^2 + delta dy^2: a sum of two non-negative
// terms.  (Summing a dx^2 + 2 b dx dy + c dy^2 cancels far along a thin
// splat, where the terms are many thousand times the result; the FP32
// alpha there would carry percent-level errors.)  Staged: A = -a/2 log2(e),
// beta, D = -delta/2 log2(e), so p2 = A w^2 + D dy^2 with w = dx + beta dy is
// log2(e) * power and G = exp(power) = 2^p2.
// Chunks of a tile's list: TGS_RENDER_CHUNKS of TGS_RENDER_CHUNK_LEN positions,
// then TGS_RENDER_LONG_CHUNKS of twice that length, each twice as long as the
// one before it and the last taking the rest.  Most walks end within the equal
// chunks (115 positions on average in the benchmark's scenes); those of a few
// percent of the tiles run to 400-850 positions, and one workgroup over all of
// the rest was the tail of the launch.  Equal chunks to the end would launch
// several empty workgroups per tile instead (0.25 ns each).
constexpr int kChunks = TGS_RENDER_CHUNKS + TGS_RENDER_LONG_CHUNKS;

__device__ __forceinline__ uint32_t chunk_begin(int c) {
  constexpr uint32_t kEqual = TGS_RENDER_CHUNKS * TGS_RENDER_CHUNK_LEN;
  return c <= TGS_RENDER_CHUNKS ? (uint32_t)(c * TGS_RENDER_CHUNK_LEN)
                                : kEqual + 2u * TGS_RENDER_CHUNK_LEN * ((1u << (c - TGS_RENDER_CHUNKS)) - 1u);
}

// The chunk that begins at position pos > 0, or 0 when none does.
__device__ __forceinline__ int chunk_at(uint32_t pos) {
  if (pos % TGS_RENDER_CHUNK_LEN != 0) return 0;
  if (pos <= (uint32_t)(TGS_RENDER_CHUNKS * TGS_RENDER_CHUNK_LEN)) return (int)(pos / TGS_RENDER_CHUNK_LEN);
#pragma unroll
  for (int c = TGS_RENDER_CHUNKS + 1; c < kChunks; ++c)
    if (pos == chunk_begin(c)) return c;
  return 0;
}

constexpr float kLog2e = 1.4426950408889634f;
constexpr int kUnroll = 8;   // forward: alphas evaluated per group
constexpr int kUnrollB = 2;  // density back-projection

__device__ __forceinline__ float splat_exponent(float dx, float dy, float A, float beta, float D) {
#pragma clang fp contract(off)
  const float w = __builtin_fmaf(beta, dy, dx);
  const float ww = w * w, yy = dy * dy;
  return __builtin_fmaf(A, ww, D * yy);
}

// alpha = min(alpha_max, o G); ok = exponent <= 0 and alpha >= alpha_min.
__device__ __forceinline__ float splat_alpha(float p2, float opacity, float amax, float& G) {
  G = __builtin_amdgcn_exp2f(p2);
  return __builtin_amdgcn_fmed3f(opacity * G, 0.f, amax);  // o G >= 0
}

__device__ __forceinline__ float one_minus_times(float T, float alpha) {
#pragma clang fp contract(off)
  return T * (1.0f - alpha);
}

struct PixelSlot {
  int loc;      // local index in the tile, -1 if none
  bool inside;  // pixel exists and lies in the image
  int64_t out;  // output index
};

template <int kBlock, bool kDense>
__device__ __forceinline__ PixelSlot pixel_of(const RasterArgs& a, int slot, int tile, int tid) {
  PixelSlot p;
  const int tx = tile % a.tiles_x, ty = tile / a.tiles_x;
  if (kDense) {
    p.loc = tid;
    const int x = tx * kTile + (tid & 15), y = ty * kTile + (tid >> 4);
    p.inside = x < a.width && y < a.height;
    p.out = (int64_t)y * a.width + x;
  } else {
    const int p0 = a.tile_off[slot], np = a.tile_off[slot + 1] - p0;
    p.loc = tid < np ? (int)a.pix[p0 + tid] : -1;
    p.inside = p.loc >= 0;
    p.out = p0 + tid;
  }
  return p;
}

// Staging of one batch: every thread holds one Gaussian of the batch in
// registers; the next batch's loads are issued before the current batch is
// evaluated, so their latency overlaps the compute.
struct Staged {
  float4 geo;  // tile-local centre x, y; staged A, beta
  float4 app;  // staged D, opacity, r, g
  float4 con;  // conic a, b, c in natural units, blue (backward only)
  float blue;
  uint32_t gid;
};

__device__ __forceinline__ Staged stage_load(const RasterArgs& a, uint32_t gid, float x0, float y0) {
#pragma clang fp contract(off)
  const float4 p0 = a.splat[3 * gid], p1 = a.splat[3 * gid + 1], p2 = a.splat[3 * gid + 2];
  Staged st;
  // exact integer difference first, then the fraction: the tile-local centre
  // keeps full FP32 precision relative to the pixel offsets
  st.geo = make_float4((p0.x - x0) + p0.z, (p0.y - y0) + p0.w, p1.x * (-0.5f * kLog2e), p1.y);
  st.app = make_float4(p1.z * (-0.5f * kLog2e), p1.w, p2.x, p2.y);
  const float b = p1.y * p1.x;  // b = beta a, c = delta + beta b
  st.con = make_float4(p1.x, b, __builtin_fmaf(p1.y, b, p1.z), p2.z);
  st.blue = p2.z;
  st.gid = gid;
  return st;
}

template <int kBlock, bool kDense>
__device__ __forceinline__ void render_fwd_view(const RasterArgs& a, float4* __restrict__ out,
                                                uint32_t* __restrict__ ncontrib,
                                                unsigned long long* __restrict__ counters,
                                                float4* __restrict__ state) {
  __shared__ float4 s_geo[kBlock];
  __shared__ float4 s_app[kBlock];
  __shared__ float s_blue[kBlock];
  if (a.mode == 2 && blockIdx.x >= *a.cont_count) return;  // workgroup-uniform
  const int slot = a.mode == 2 ? (int)a.cont_list[blockIdx.x] : (int)blockIdx.x, tid = threadIdx.x;
  const int tile = kDense ? slot : a.valid_tiles[slot];
  const int tx = tile % a.tiles_x, ty = tile / a.tiles_x;
  const PixelSlot px = pixel_of<kBlock, kDense>(a, slot, tile, tid);
  const float lx = (float)(px.loc & 15), ly = (float)(px.loc >> 4);
  const float x0 = (float)(tx * kTile), y0 = (float)(ty * kTile);
  const TileList L = tile_list(a, tile);
  const uint2 range = make_uint2(0u, L.len);
  const float amin = a.alpha_min, amax = a.alpha_max, tmin = a.T_min;

  float T = 1.f, c0 = 0.f, c1 = 0.f, c2 = 0.f;
  uint32_t last = 0;
  uint32_t n_blend = 0;  // this lane's blends (summed over the wave at the end)
  // a pixel that has stopped, or is none, compares its alphas with a NaN: one
  // register in place of a lane mask in every test.  The walk is bound by issue,
  // and a third of it was scalar: with masks for done and stopped pixels and
  // counted evaluations 1296x840 dense took 126 us (300k Gaussians) and 199 us
  // (1600x1060, 1.5M), now 107 and 166; a quarter of the pixels 66, now 58.
  // Counting with scalar popcounts instead: 125 us.
  float amin_l = px.inside ? amin : __builtin_nanf("");
  auto is_done = [&] { return amin_l != amin_l; };
  uint32_t stop_at = 0;  // list position of the T_min stop

  // prologue: records of batch 0 and ids of batch 1 in flight
  Staged nxt = {};
  uint32_t g_after = 0;
  if (range.x + tid < range.y) nxt = stage_load(a, list_id(a, L, range.x + tid), x0, y0);
  if (range.x + kBlock + tid < range.y) g_after = list_id(a, L, range.x + kBlock + tid);

  for (uint32_t start = range.x; start < range.y; start += kBlock) {
    if (__syncthreads_count(is_done()) == kBlock) break;
    const bool live = start + tid < range.y;  // past the range: a zero-opacity record
    s_geo[tid] = live ? nxt.geo : make_float4(0.f, 0.f, 0.f, 0.f);
    s_app[tid] = live ? nxt.app : make_float4(0.f, 0.f, 0.f, 0.f);
    s_blue[tid] = live ? nxt.blue : 0.f;
    __syncthreads();
    const uint32_t i1 = start + kBlock + tid, i2 = start + 2 * kBlock + tid;
    if (i1 < range.y) nxt = stage_load(a, g_after, x0, y0);
    if (i2 < range.y) g_after = list_id(a, L, i2);
    const int cnt = (int)min((uint32_t)kBlock, range.y - start);
    const uint32_t pos0 = start - range.x;
    // groups of kUnroll Gaussians: their alphas are independent and are
    // evaluated first, then composited in order (entries past cnt hold a
    // zero-opacity record and never composite)
    for (int j = 0; j < cnt; j += kUnroll) {
      if (ballot(!is_done()) == 0ull) break;  // the whole wave has terminated
      const uint32_t pos = pos0 + (uint32_t)j;  // uniform; chunk starts are multiples of kUnroll
      if (state != nullptr) {
        const int c = chunk_at(pos);  // uniform
        if (c > 0) state[((int64_t)slot * (kChunks - 1) + c - 1) * kBlock + tid] = make_float4(T, c0, c1, c2);
      }
      float al[kUnroll], pw[kUnroll], cr[kUnroll], cg[kUnroll], cb[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const float4 ge = s_geo[j + u];
        const float4 ap = s_app[j + u];
        pw[u] = splat_exponent(lx - ge.x, ly - ge.y, ge.z, ge.w, ap.x);
        float G;
        al[u] = splat_alpha(pw[u], ap.y, amax, G);
        cr[u] = ap.z;
        cg[u] = ap.w;
        cb[u] = s_blue[j + u];
      }
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const float t_next = one_minus_times(T, al[u]);
        const bool hit = pw[u] <= 0.f && al[u] >= amin_l;
        const bool stop = hit && t_next < tmin, ok = hit && !stop;
        stop_at = stop ? pos0 + (uint32_t)(j + u) : stop_at;
        amin_l = stop ? __builtin_nanf("") : amin_l;
        const float w = ok ? al[u] * T : 0.f;
        c0 = __builtin_fmaf(w, cr[u], c0);
        c1 = __builtin_fmaf(w, cg[u], c1);
        c2 = __builtin_fmaf(w, cb[u], c2);
        T = ok ? t_next : T;
        last = ok ? pos0 + (uint32_t)(j + u) + 1u : last;
        n_blend += ok ? 1u : 0u;
      }
    }
  }
  const bool stopped = px.inside && is_done();
  // evaluations: every list position up to and with the stop
  uint32_t n_eval = !px.inside ? 0u : (stopped ? stop_at + 1u : L.len);
  if (px.inside) {
    out[px.out] = make_float4(c0 + T * a.bg0, c1 + T * a.bg1, c2 + T * a.bg2, T);
    ncontrib[px.out] = last;
  }
  if (a.mode == 1) {
    // a pixel that ran off its list without stopping needs the continuation;
    // its counts come from the continuation pass
    const bool open = px.inside && !stopped;
    if (open) n_eval = n_blend = 0u;
    if (ballot(open) != 0ull && lane_id() == 0 &&
        atomicCAS(&a.cont_slot[tile], -1, slot) == -1)  // the tile's first marking wave lists it
      a.cont_list[atomicAdd(a.cont_count, 1u)] = (uint32_t)slot;
  } else if (a.mode == 2 && stopped && stop_at < L.n1) {
    n_eval = n_blend = 0u;  // stopped within the prefix: counted by the prefix pass
  }
  if (counters != nullptr) {
    n_eval = (uint32_t)wave_sum_i((int)n_eval);
    n_blend = (uint32_t)wave_sum_i((int)n_blend);
  }
  if (counters != nullptr && lane_id() == 0) {  // wave totals
    const int cs = blockIdx.x & (TGS_COUNTER_SLOTS - 1);
    atomicAdd(&counters[cs], (unsigned long long)n_eval);
    atomicAdd(&counters[TGS_COUNTER_SLOTS + cs], (unsigned long long)n_blend);
  }
}

// The views of a step in one launch, view k in grid layer z = k: a small view
// has fewer workgroups than the device holds.  Four 256x256 views of 64 tiles
// each take 39 us together, 4 x 36 us one by one (the backward 15 us, 4 x 12).
struct FwdArgs {
  RasterArgs a;
  float4* out;
  uint32_t* ncontrib;
  unsigned long long* counters;
  float4* state;
  int grid;  // the view's workgroups; the launch's grid is the largest view's
};

template <int kBlock, bool kDense>
__global__ void __launch_bounds__(kBlock) render_fwd_kernel(Batch<FwdArgs> b) {
  const FwdArgs& v = b.v[blockIdx.z];
  if ((int)blockIdx.x >= v.grid) return;
  render_fwd_view<kBlock, kDense>(v.a, v.out, v.ncontrib, v.counters, v.state);
}

__device__ __forceinline__ float swap_sum32(float x, float y) {
  // after the swap x = [x_lo | y_lo], y = [x_hi | y_hi]: the sum folds both
  // values to 32 lanes, x in lanes 0-31 and y in lanes 32-63
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ float swap_sum16(float x, float y) {
  // rows of 16 lanes: x = [x0 y0 x2 y2], y = [x1 y1 x3 y3] after the swap
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ float row_sum16(float v) {
  v += dpp_f<kDppQuadPerm1032>(0.f, v);
  v += dpp_f<kDppQuadPerm2301>(0.f, v);
  v += dpp_f<kDppRowHalfMirror>(0.f, v);
  v += dpp_f<kDppRowMirror>(0.f, v);
  return v;  // every lane of a row holds the row's sum
}

// Sum over the quads of a row of 16 lanes: every lane ends with the sum over
// the row's lanes of its own index modulo 4.
__device__ __forceinline__ float row_sum_quads(float v) {
  v += dpp_f<0x128>(0.f, v);  // row_ror:8
  v += dpp_f<0x124>(0.f, v);  // row_ror:4
  return v;
}

// Optional density-control sums in the backward (Sec. 3.8): the replay
// already has each composited Gaussian's weight w = T alpha and each lane's
// own centre gradient.
struct DensityArgs {
  const float* err;  // [P] per-pixel error e(p), indexed like out
  float* stats;      // [n][4] E, W, D, sum of per-pixel NDC centre-gradient norms (+=)
  int64_t n;
};

// The backward's sums over pixels.
//
// Per (Gaussian, pixel) the replay leaves two scalars, q = dL/d opacity at
// that pixel (G dalpha where alpha is not clamped) and the weight w.  With d =
// the pixel's offset from the centre, every gradient of the Gaussian is a
// moment of q or w over the pixels: sum q, sum q d, sum q d d^T and sum w g
// (g = dL/d colour of the pixel).  Summing nine values across a wave with
// lane swaps and DPP adds takes ~40 of the ~83 vector instructions of a
// (Gaussian, wave) step, and the walk is bound by vector issue.  Instead q and
// w of four Gaussians go, through LDS private to the wave (whose LDS
// operations execute in order), from a lane per pixel to a lane per Gaussian
// and four pixels.  There a lane sums the moments of q over its four pixels,
// each product formed per pixel from that pixel's own offset and each moment
// in a sum of its own, and the colour sums run on the matrix cores as 4
// Gaussians x 64 pixels times 64 pixels x 4 columns (v_mfma_f32_4x4x1, 16
// blocks, one pixel per block and instruction, FP32 products and sums).  Lane
// swaps and row rotations fold the 16 lanes (or blocks) of a Gaussian into a
// table; at the end of a batch a thread per Gaussian combines its row (over
// the workgroup's waves, in wave order) and consecutive lanes add the nine
// gradients of consecutive Gaussians (36-byte runs).
// 300k Gaussians, 1296 x 840: 73 us at 64 samples per tile and 214 us dense,
// with nine lane sums 89 and 274.  Moments about the tile's centre, formed with
// the columns (1, x, y) on the matrix cores and shifted to the Gaussian's
// centre after the sums, took 76 and 235 us and lost up to a factor of the
// tile's half width over |d| in precision; an overflow in one moment also
// reached the others of its matrix.
constexpr int kBwdBatch = TGS_RENDER_CHUNK_LEN;  // Gaussians per batch: one short chunk
constexpr int kBwdGroup = 4;                     // Gaussians per matrix
constexpr int kBwdStage = 2 * kBwdBatch;         // Gaussians loaded per round
static_assert(kBwdBatch == 32, "a round's composited Gaussians are kept as a 32-bit mask");

typedef float v4f __attribute__((ext_vector_type(4)));

// Sums of the four rows (Gaussians) of a 16-block accumulator over the
// blocks: row r of 16 lanes holds Gaussian ((r & 1) << 1) | (r >> 1), lane l
// of the row column l % 4.
__device__ __forceinline__ float block_sums(const v4f& c) {
  return row_sum_quads(swap_sum16(swap_sum32(c[0], c[1]), swap_sum32(c[2], c[3])));
}

// Two 4 Gaussians x 64 pixels matrices from a lane per pixel (x[u], y[u]:
// Gaussian u) to the operands of the four instructions s: lane l gets
// Gaussian l % 4 of pixel 16 s + l / 4.  The buffer is the wave's own and its
// LDS operations execute in order, so the writes of one call follow the reads
// of the call before it.
template <typename F>
__device__ __forceinline__ void transpose2(float* tr, int lane, const float (&x)[4], const float (&y)[4], F&& f) {
  float4* tw = reinterpret_cast<float4*>(tr);
  tw[lane] = make_float4(x[0], x[1], x[2], x[3]);
  tw[kWave + lane] = make_float4(y[0], y[1], y[2], y[3]);
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  float xs[4], ys[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    xs[s] = tr[s * kWave + lane];
    ys[s] = tr[(4 + s) * kWave + lane];
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int s = 0; s < 4; ++s) f(s, xs[s], ys[s]);
}

// kDet: the deterministic variant.  Instead of adding the pair's nine sums to
// g2d[gid] with atomics, it stores them to g2d[pos * 9] (g2d is then the
// partial buffer, pos the pair's index in the sorted list);
// det_reduce_kernel adds them up per Gaussian in a fixed order.
template <int kBlock, bool kDense, bool kDensity = false, bool kDet = false>
__device__ __forceinline__ void render_bwd_view(const RasterArgs& a, const float4* __restrict__ out,
                                                const uint32_t* __restrict__ ncontrib,
                                                const float4* __restrict__ dL, float* __restrict__ g2d,
                                                const float4* __restrict__ state, uint8_t* __restrict__ touched,
                                                const DensityArgs& dens) {
  constexpr int kWaves = kBlock / kWave;
  constexpr int kCols = kDensity ? 16 : 12; // sums per Gaussian in the table
  constexpr int kFields = kDensity ? 13 : 9;
  __shared__ float4 s_geo[kBwdStage];
  __shared__ float4 s_app[kBwdStage];
  __shared__ float4 s_con[kBwdStage];  // conic a, b, c (natural units), blue
  __shared__ uint32_t s_gid[kBwdStage];
  // a wave's transposition buffer (two matrices at a time); before the walk its pixels' columns
  __shared__ __align__(16) float s_tr[kWaves][2][kWave * kBwdGroup];
  __shared__ __align__(16) float s_tab[kWaves][kBwdBatch * kCols];
  __shared__ uint32_t s_hit[kWaves];  // Gaussians of the batch composited in the wave
  // the last chunks (the longest walks) are dispatched first, so their
  // workgroups run beside the short ones
  const int slot = blockIdx.x, chunk = (int)gridDim.y - 1 - (int)blockIdx.y, tid = threadIdx.x;
  const int lane = lane_id(), wave = tid / kWave;
  const int tile = kDense ? slot : a.valid_tiles[slot];
  const int tx = tile % a.tiles_x, ty = tile / a.tiles_x;
  const TileList L = tile_list(a, tile);
  const uint2 range = make_uint2(0u, L.len);
  // list positions [begin, end) of this chunk (one chunk without a state record)
  const uint32_t begin = range.x + chunk_begin(chunk);
  if (begin >= range.y && chunk > 0) return;  // workgroup-uniform
  const uint32_t end =
      chunk + 1 == (int)gridDim.y ? range.y : min(range.y, range.x + chunk_begin(chunk + 1));
  // a thread of the first 64 stages one Gaussian; the ids of the next round
  // are loaded ahead, the records are not (holding them over the walk costs
  // the registers of a wave per SIMD).  The first ids are asked for here,
  // beside the pixels' contributor counts.
  const bool stager = tid < kBwdStage;
  uint32_t g_next = 0;
  if (stager && begin + tid < end) g_next = list_id(a, L, begin + tid);
  const PixelSlot px = pixel_of<kBlock, kDense>(a, slot, tile, tid);
  const float lx = (float)(px.loc & 15), ly = (float)(px.loc >> 4);
  const float x0 = (float)(tx * kTile), y0 = (float)(ty * kTile);
  const float amin = a.alpha_min, amax = a.alpha_max;
  const float hw = 0.5f * (float)a.width, hh = 0.5f * (float)a.height;  // pixel -> NDC units

  float Cout0 = 0.f, Cout1 = 0.f, Cout2 = 0.f, g0 = 0.f, g1 = 0.f, g2 = 0.f;
  uint32_t last = 0;
  float e_pix = 0.f;
  if (px.inside) last = ncontrib[px.out];
  // positions below lim are this chunk's and at or before the pixel's last
  // composited one
  const uint32_t lim = min(last, end - range.x);
  const bool done = last <= begin - range.x;  // nothing composited from this chunk on
  // a chunk past every pixel's last composited position has nothing to do:
  // it leaves before reading the pixels' outputs, gradients and state
  if (__syncthreads_count(done) == kBlock) return;
  if (px.inside) {
    const float4 o = out[px.out];
    const float4 d = dL[px.out];
    Cout0 = o.x; Cout1 = o.y; Cout2 = o.z;
    g0 = d.x; g1 = d.y; g2 = d.z;
    if (kDensity) e_pix = dens.err[px.out];
  }
  // T and S = sum_c g_c (C_c - acc_c): the loss-weighted colour behind the
  // current Gaussian (final colour minus what is composited in front of
  // and at it), updated as S -= w * sum_c g_c colour_c
  float T = 1.f, acc0 = 0.f, acc1 = 0.f, acc2 = 0.f;
  if (chunk > 0 && !done) {
    const float4 st = state[((int64_t)slot * (kChunks - 1) + chunk - 1) * kBlock + tid];
    T = st.x;
    acc0 = st.y;
    acc1 = st.z;
    acc2 = st.w;
  }
  float S = g0 * (Cout0 - acc0) + g1 * (Cout1 - acc1) + g2 * (Cout2 - acc2);

  auto stage = [&](uint32_t start) {
    Staged st = {};
    if (start + tid < end) st = stage_load(a, g_next, x0, y0);
    if (start + kBwdStage + tid < end) g_next = list_id(a, L, start + kBwdStage + tid);
    s_geo[tid] = st.geo;
    s_app[tid] = st.app;
    s_con[tid] = st.con;
    s_gid[tid] = st.gid;
  };
  if (stager) stage(begin);

  // the pixels as the sums take them: lane l's are 16 s + l / 4, s = 0 .. 3;
  // their positions, and as a matrix operand column l % 4 of their colour gradients
  float* const tr = &s_tr[wave][0][0];
  float* const s_fin = &s_tr[0][0][0];  // the batch's gradients, after the walk
  static_assert(kBwdBatch * kFields <= 2 * kWave * kBwdGroup, "the gradients fit one wave's buffer");
  {
    float4* row = reinterpret_cast<float4*>(tr);
    row[2 * lane] = make_float4(lx, ly, 0.f, 0.f);
    row[2 * lane + 1] = make_float4(g0, g1, g2, e_pix);
  }
  __syncthreads();
  const int sub = lane & 3;  // the lane's Gaussian of a group, and its column
  float xs[4], ys[4], bw[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const float* row = tr + (16 * s + (lane >> 2)) * 8;
    xs[s] = row[0];
    ys[s] = row[1];
    bw[s] = row[4 + sub];
  }

  for (uint32_t start = begin; start < end; start += kBwdBatch) {
    if (__syncthreads_count(lim <= start - range.x) == kBlock) break;
    const int st0 = (int)((start - begin) & (uint32_t)(kBwdStage - 1));  // the batch's first staged entry
    if (st0 == 0 && start != begin) {
      if (stager) stage(start);
      __syncthreads();
    }
    const float4* const b_geo = s_geo + st0;
    const float4* const b_app = s_app + st0;
    const float4* const b_con = s_con + st0;
    const uint32_t* const b_gid = s_gid + st0;
    const int cnt = (int)min((uint32_t)kBwdBatch, end - start);
    const uint32_t pos0 = start - range.x;
    uint32_t hit = 0;  // wave-uniform
    for (int j = 0; j < cnt; j += kBwdGroup) {
      if (ballot(pos0 + (uint32_t)j < lim) == 0ull) break;  // the whole wave has finished
      float q[4], w[4];
      uint32_t some = 0;
#pragma unroll
      for (int u = 0; u < kBwdGroup; ++u) {
        const float4 ge = b_geo[j + u];
        const float4 ap = b_app[j + u];
        const float blue = b_con[j + u].w;
        const float dx = lx - ge.x, dy = ly - ge.y;
        const float p2 = splat_exponent(dx, dy, ge.z, ge.w, ap.x);
        float G;
        const float alpha = splat_alpha(p2, ap.y, amax, G);
        const bool ok = pos0 + (uint32_t)(j + u) < lim && p2 <= 0.f && alpha >= amin;
        w[u] = ok ? alpha * T : 0.f;
        // loss-weighted colour of this Gaussian: sum_c g_c colour_c
        const float gc = __builtin_fmaf(g2, blue, __builtin_fmaf(g1, ap.w, g0 * ap.z));
        const float T_before = T;
        T = ok ? one_minus_times(T, alpha) : T;
        S = __builtin_fmaf(-w[u], gc, S);
        const float inv = __builtin_amdgcn_rcpf(1.f - alpha);
        // dL/dalpha = T_before sum_c g_c colour_c - S / (1 - alpha)
        const float dalpha = __builtin_fmaf(T_before, gc, -S * inv);
        q[u] = ok && ap.y * G < amax ? G * dalpha : 0.f;  // clamped alphas pass nothing
        some |= __builtin_amdgcn_ballot_w64(ok) != 0ull ? 1u << u : 0u;
      }
      if (some == 0u) continue;  // wave-uniform: no pixel of the wave composited any of the four
      hit |= some << j;
      const float4 ge = b_geo[j + sub];
      v4f mc = {0.f, 0.f, 0.f, 0.f};
      float m0 = 0.f, mx = 0.f, my = 0.f, mxx = 0.f, mxy = 0.f, myy = 0.f;
      float mw = 0.f, md = 0.f, mn = 0.f;  // density: w, w D and the norm of the pixel's own centre gradient
      transpose2(tr, lane, q, w, [&](int s, float qs, float ws) {
        const float dx = xs[s] - ge.x, dy = ys[s] - ge.y;
        const float qx = qs * dx, qy = qs * dy;
        m0 += qs;
        mx += qx;
        my += qy;
        mxx = __builtin_fmaf(qx, dx, mxx);
        mxy = __builtin_fmaf(qx, dy, mxy);
        myy = __builtin_fmaf(qy, dy, myy);
        mc = __builtin_amdgcn_mfma_f32_4x4x1f32(ws, bw[s], mc, 0, 0, 0);
        if constexpr (kDensity) {
          // D = the distance, sqrt(-2 power); correctly rounded roots, as in the walk of its own below
          constexpr float kTwoLn2 = 1.3862943611198906f;
          const float4 ap = b_app[j + sub], cn = b_con[j + sub];
          const float p2 = splat_exponent(dx, dy, ge.z, ge.w, ap.x);
          const float dist = __builtin_sqrtf(fmaxf(-kTwoLn2 * p2, 0.f));
          const float nx = hw * ((cn.x * dx + cn.y * dy) * (ap.y * qs));
          const float ny = hh * ((cn.y * dx + cn.z * dy) * (ap.y * qs));
          mw += ws;
          md += ws > 0.f ? dist * ws : 0.f;
          mn += __builtin_sqrtf(nx * nx + ny * ny);
        }
      });
      // four values per register and row of 16 lanes; the colours' rows are Gaussians, the others' the values
      const float r0 = row_sum_quads(swap_sum16(swap_sum32(mx, my), swap_sum32(mxx, mxy)));
      const float r1 = row_sum_quads(swap_sum16(swap_sum32(myy, m0), kDensity ? swap_sum32(mw, md) : 0.f));
      const float r2 = block_sums(mc);
      const int quad = (lane >> 2) & 3, row = lane >> 4, in = ((row & 1) << 1) | (row >> 1);
      float val = quad == 0 ? r0 : (quad == 1 ? r1 : r2);
      if constexpr (kDensity) {
        const float r3 = row_sum_quads(swap_sum16(swap_sum32(mn, 0.f), 0.f));
        val = quad == 3 ? r3 : val;
      }
      if (kDensity || quad < 3)
        s_tab[wave][(j + (quad == 2 ? in : sub)) * kCols + quad * 4 + (quad == 2 ? sub : in)] = val;
    }
    if (lane == 0) s_hit[wave] = hit;
    __syncthreads();
    uint32_t any = 0;
#pragma unroll
    for (int v = 0; v < kWaves; ++v) any |= s_hit[v];
    if (any == 0u) continue;  // workgroup-uniform
    if (tid < kBwdBatch && (any >> tid) & 1u) {
      // row of the table: sum q dx, q dy, q dx dx, q dx dy; q dy dy, q, (density)
      // w, w D; w g0, w g1, w g2, w e; |n|, -, -, -
      float t[kCols];
#pragma unroll
      for (int k = 0; k < kCols; ++k) t[k] = 0.f;
#pragma unroll
      for (int v = 0; v < kWaves; ++v) {
        if (!((s_hit[v] >> tid) & 1u)) continue;
        const float4* tb = reinterpret_cast<const float4*>(&s_tab[v][tid * kCols]);
#pragma unroll
        for (int k = 0; k < kCols / 4; ++k) {
          const float4 x = tb[k];
          t[4 * k] += x.x;
          t[4 * k + 1] += x.y;
          t[4 * k + 2] += x.z;
          t[4 * k + 3] += x.w;
        }
      }
      const float4 cn = b_con[tid];
      const float opac = b_app[tid].y;
      float* fin = s_fin + tid * kFields;
      fin[0] = opac * __builtin_fmaf(cn.x, t[0], cn.y * t[1]);
      fin[1] = opac * __builtin_fmaf(cn.y, t[0], cn.z * t[1]);
      fin[2] = -0.5f * opac * t[2];
      fin[3] = -opac * t[3];
      fin[4] = -0.5f * opac * t[4];
      fin[5] = t[5];
      fin[6] = t[8];
      fin[7] = t[9];
      fin[8] = t[10];
      if constexpr (kDensity) {
        fin[9] = t[11];
        fin[10] = t[6];
        fin[11] = t[7];
        fin[12] = t[12];
      }
      if (touched != nullptr) touched[b_gid[tid]] = 1u;  // composited at a sample
    }
    __syncthreads();
    int e0 = tid;
    asm volatile("" : "+v"(e0));  // keeps the entries' indices out of the registers that live over the walk
#pragma unroll 1
    for (int e = e0; e < kBwdBatch * kFields; e += kBlock) {
      const int k = e / kFields, f = e - k * kFields;
      if (!((any >> k) & 1u)) continue;
      const float val = s_fin[e];
      const uint32_t gid = b_gid[k];
      if constexpr (kDet) {
        // the pair's index in vals (the deterministic backward takes single-segment lists)
        g2d[(size_t)(L.b1 + start + (uint32_t)k) * 9 + (size_t)f] = val;
      } else if (val != 0.f) {
        if (!kDensity || f < 9) unsafeAtomicAdd(&g2d[(size_t)gid * 9 + (size_t)f], val);
        else if (gid < (uint32_t)dens.n) unsafeAtomicAdd(&dens.stats[(size_t)gid * 4 + (size_t)(f - 9)], val);
      }
    }
  }
}

struct BwdArgs {
  RasterArgs a;
  const float4* out;
  const uint32_t* ncontrib;
  const float4* dL;
  float* g2d;
  const float4* state;
  uint8_t* touched;
  DensityArgs dens;
  int grid;  // as in FwdArgs
};

template <int kBlock, bool kDense, bool kDensity, bool kDet>
__global__ void __launch_bounds__(kBlock, kBlock == 64 ? 6 : 5) render_bwd_kernel(Batch<BwdArgs> b) {
  const BwdArgs& v = b.v[blockIdx.z];
  if ((int)blockIdx.x >= v.grid) return;
  render_bwd_view<kBlock, kDense, kDensity, kDet>(v.a, v.out, v.ncontrib, v.dL, v.g2d, v.state, v.touched, v.dens);
}

// Back-projection of per-pixel statistics onto the Gaussians (Sec. 3.8,
// Eq. gauss_err_accum): the forward walk is replayed with the same alpha
// decisions, bounded by the forward's contributor count, and every
// composited Gaussian collects e(p) w, w and D(p) w with w = T alpha and
// D(p) = sqrt(d^T Q d) = sqrt(-2 ln2 p2) (p2 is the staged exponent, log2(e)
// times the power).  Per Gaussian the three values are summed across the
// wave (lane-half swaps, then DPP within rows of 16) and three lanes issue
// one float atomic each into stats[gid][0 | 1 | 2] (one 16-byte slot, so the
// three atomics touch one cache line).  With the forward's
// state record the walk is split into chunks exactly as the backward's.
template <int kBlock, bool kDense>
__global__ void __launch_bounds__(kBlock) render_accum_kernel(RasterArgs a, const uint32_t* __restrict__ ncontrib,
                                                              const float* __restrict__ err, int64_t n,
                                                              float* __restrict__ stats,
                                                              const float4* __restrict__ state) {
  __shared__ float4 s_geo[kBlock];
  __shared__ float s_opa[kBlock];
  __shared__ float s_cc[kBlock];
  __shared__ uint32_t s_gid[kBlock];
  // the last chunks (the longest walks) are dispatched first, so their
  // workgroups run beside the short ones
  const int slot = blockIdx.x, chunk = (int)gridDim.y - 1 - (int)blockIdx.y, tid = threadIdx.x;
  const int tile = kDense ? slot : a.valid_tiles[slot];
  const int tx = tile % a.tiles_x, ty = tile / a.tiles_x;
  const TileList L = tile_list(a, tile);
  const uint2 range = make_uint2(0u, L.len);
  const uint32_t begin = range.x + chunk_begin(chunk);
  if (begin >= range.y && chunk > 0) return;  // workgroup-uniform
  const uint32_t end =
      chunk + 1 == (int)gridDim.y ? range.y : min(range.y, range.x + chunk_begin(chunk + 1));
  const PixelSlot px = pixel_of<kBlock, kDense>(a, slot, tile, tid);
  const float lx = (float)(px.loc & 15), ly = (float)(px.loc >> 4);
  const float x0 = (float)(tx * kTile), y0 = (float)(ty * kTile);
  const float amin = a.alpha_min, amax = a.alpha_max;
  constexpr float kTwoLn2 = 1.3862943611198906f;
  // lane 0 of row 0 sums field 0, lane 0 of row 2 field 1, lane 0 of row 1 field 2
  const int lane = lane_id();
  const int field = (lane & 15) != 0 ? -1 : (lane == 0 ? 0 : (lane == 32 ? 1 : (lane == 16 ? 2 : -1)));

  float e = 0.f;
  uint32_t last = 0;
  if (px.inside) {
    e = err[px.out];
    last = ncontrib[px.out];
  }
  bool done = last <= begin - range.x;  // nothing composited from this chunk on
  float T = 1.f;
  if (chunk > 0 && !done) T = state[((int64_t)slot * (kChunks - 1) + chunk - 1) * kBlock + tid].x;

  Staged nxt = {};
  uint32_t g_after = 0;
  if (begin + tid < end) nxt = stage_load(a, list_id(a, L, begin + tid), x0, y0);
  if (begin + kBlock + tid < end) g_after = list_id(a, L, begin + kBlock + tid);

  for (uint32_t start = begin; start < end; start += kBlock) {
    if (__syncthreads_count(done) == kBlock) break;
    const bool live = start + tid < end;
    s_geo[tid] = live ? nxt.geo : make_float4(0.f, 0.f, 0.f, 0.f);
    s_cc[tid] = live ? nxt.app.x : 0.f;
    s_opa[tid] = live ? nxt.app.y : 0.f;
    s_gid[tid] = nxt.gid;
    __syncthreads();
    const uint32_t i1 = start + kBlock + tid, i2 = start + 2 * kBlock + tid;
    if (i1 < end) nxt = stage_load(a, g_after, x0, y0);
    if (i2 < end) g_after = list_id(a, L, i2);
    const int cnt = (int)min((uint32_t)kBlock, end - start);
    const uint32_t pos0 = start - range.x;
    for (int j = 0; j < cnt; j += kUnrollB) {
      if (__ballot(!done) == 0ull) break;  // the whole wave has finished
      float al[kUnrollB], pw[kUnrollB];
#pragma unroll
      for (int u = 0; u < kUnrollB; ++u) {
        const float4 ge = s_geo[j + u];
        pw[u] = splat_exponent(lx - ge.x, ly - ge.y, ge.z, ge.w, s_cc[j + u]);
        float G;
        al[u] = splat_alpha(pw[u], s_opa[j + u], amax, G);
      }
#pragma unroll
      for (int u = 0; u < kUnrollB; ++u) {
        if (j + u >= cnt) break;  // uniform
        const bool ok = !done && pw[u] <= 0.f && al[u] >= amin;
        const float w = ok ? al[u] * T : 0.f;
        T = ok ? one_minus_times(T, al[u]) : T;
        done = done || (pos0 + (uint32_t)(j + u) + 1u >= last);
        if (__ballot(ok) != 0ull) {
          const float dist = __builtin_sqrtf(fmaxf(-kTwoLn2 * pw[u], 0.f));
          const float p01 = swap_sum32(e * w, w);
          const float p2 = swap_sum32(dist * w, 0.f);
          float r = row_sum16(swap_sum16(p01, p2));
          asm volatile("" : "+v"(r));  // the whole row sum with the whole wave active
          const uint32_t gid = __builtin_amdgcn_readfirstlane(s_gid[j + u]);  // uniform
          if (field >= 0 && r != 0.f && gid < (uint32_t)n) unsafeAtomicAdd(&stats[(int64_t)gid * 4 + field], r);
        }
      }
    }
  }
}

template <int kBlock, bool kDense>
static void launch_fwd(const Batch<FwdArgs>& b, int views, int grid, hipStream_t s) {
  hipLaunchKernelGGL((render_fwd_kernel<kBlock, kDense>), dim3((unsigned)grid, 1, (unsigned)views), dim3(kBlock), 0, s,
                     b);
}

// One chunk per tile without the forward's state record, of any view.
template <int kBlock, bool kDense, bool kDet>
static void launch_bwd(const Batch<BwdArgs>& b, int views, int grid, bool density, hipStream_t s) {
  const dim3 g((unsigned)grid, b.v[0].state != nullptr ? kChunks : 1, (unsigned)views);
  if constexpr (kDet)
    hipLaunchKernelGGL((render_bwd_kernel<kBlock, kDense, false, true>), g, dim3(kBlock), 0, s, b);
  else if (density)
    hipLaunchKernelGGL((render_bwd_kernel<kBlock, kDense, true, false>), g, dim3(kBlock), 0, s, b);
  else
    hipLaunchKernelGGL((render_bwd_kernel<kBlock, kDense, false, false>), g, dim3(kBlock), 0, s, b);
}

__global__ void __launch_bounds__(256) zero_f32_kernel(float* __restrict__ p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0.f;
}

// Deterministic reduction of the partial records: a thread per Gaussian
// visits the tiles of its rectangle in row-major order, finds its pair in
// the tile's list by binary search on (depth bits, id) (the list's order),
// and adds the pair's record; the total is added to g2d once.  Any order
// would do; a fixed one gives the same bits on every
// run.
__global__ void __launch_bounds__(256) det_reduce_kernel(const int4* __restrict__ rect, const float* __restrict__ depth,
                                                         const uint32_t* __restrict__ vals,
                                                         const uint2* __restrict__ ranges, int64_t n, int tiles_x,
                                                         int tiles_y, const float* __restrict__ partial,
                                                         float* __restrict__ g2d) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int4 r = rect[i];
  r.x = min(max(r.x, 0), tiles_x);
  r.z = min(max(r.z, r.x), tiles_x);
  r.y = min(max(r.y, 0), tiles_y);
  r.w = min(max(r.w, r.y), tiles_y);
  const uint32_t key = __float_as_uint(depth[i]), id = (uint32_t)i;
  float acc[9] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  bool any = false;
  for (int ty = r.y; ty < r.w; ++ty)
    for (int tx = r.x; tx < r.z; ++tx) {
      const uint2 rg = ranges[ty * tiles_x + tx];
      uint32_t lo = rg.x, hi = rg.y;
      while (lo < hi) {  // first position not below (key, id)
        const uint32_t mid = lo + (hi - lo) / 2;
        const uint32_t gm = vals[mid], km = __float_as_uint(depth[gm]);
        if (km < key || (km == key && gm < id)) lo = mid + 1;
        else hi = mid;
      }
      if (lo < rg.y && vals[lo] == id) {
        const float* p = partial + (size_t)lo * 9;
        for (int f = 0; f < 9; ++f) acc[f] += p[f];
        any = true;
      }
    }
  if (any)
    for (int f = 0; f < 9; ++f) g2d[i * 9 + f] += acc[f];
}

// Workgroup size of the raster kernels for a launch.
static int raster_block(bool dense, int32_t max_per_tile) {
  if (dense || max_per_tile > 128) return 256;
  return max_per_tile <= 64 ? 64 : 128;
}

static int32_t make_args(const float* splat, const uint32_t* vals, const uint32_t* ranges,
                         int32_t tiles_x, int32_t tiles_y, int32_t width, int32_t height,
                         const int32_t* valid_tiles, const int32_t* tile_off, const uint8_t* pix,
                         int32_t n_st, int32_t max_per_tile, const tgs_raster_params* rp,
                         const char* who, RasterArgs& a) {
  TGS_REQUIRE(rp != nullptr, "%s: null raster params", who);
  TGS_REQUIRE(width > 0 && height > 0 && tiles_x == (int32_t)ceil_div(width, kTile) &&
                  tiles_y == (int32_t)ceil_div(height, kTile),
              "%s: tile grid %d x %d does not match image %d x %d", who, tiles_x, tiles_y, width,
              height);
  TGS_REQUIRE(splat && vals && ranges, "%s: null splat/vals/ranges", who);
  TGS_REQUIRE(((uintptr_t)splat & 15) == 0, "%s: splat must be 16-byte aligned", who);
  if (valid_tiles != nullptr) {
    TGS_REQUIRE(tile_off && pix, "%s: null tile_off/pix", who);
    TGS_REQUIRE(n_st >= 0 && (int64_t)n_st <= (int64_t)tiles_x * tiles_y, "%s: bad n_st %d", who, n_st);
    TGS_REQUIRE(max_per_tile >= 0 && max_per_tile <= kTilePixels, "%s: bad max_per_tile %d", who,
                max_per_tile);
  }
  a.splat = (const float4*)splat;
  a.vals = vals;
  a.ranges = (const uint2*)ranges;
  a.valid_tiles = valid_tiles;
  a.tile_off = tile_off;
  a.pix = pix;
  a.tiles_x = tiles_x;
  a.tiles_y = tiles_y;
  a.width = width;
  a.height = height;
  a.alpha_min = rp->alpha_min;
  a.alpha_max = rp->alpha_max;
  a.T_min = rp->T_min;
  a.bg0 = rp->bg[0];
  a.bg1 = rp->bg[1];
  a.bg2 = rp->bg[2];
  a.vals2 = nullptr;
  a.ranges2 = nullptr;
  a.mode = 0;
  a.cont_slot = nullptr;
  a.cont_list = nullptr;
  a.cont_count = nullptr;
  return TGS_OK;
}

// The second list segment of the two-segment entry points.
static int32_t set_second(RasterArgs& a, const uint32_t* vals2, const uint32_t* ranges2, const char* who) {
  TGS_REQUIRE(vals2 && ranges2, "%s: null vals2/ranges2", who);
  a.vals2 = vals2;
  a.ranges2 = (const uint2*)ranges2;
  return TGS_OK;
}

__global__ void __launch_bounds__(256) fill_i32_kernel(int32_t* __restrict__ p, int64_t n, int32_t v,
                                                       uint32_t* __restrict__ count) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
  if (i == 0 && count != nullptr) *count = 0u;
}

}  // namespace tgs

using namespace tgs;

extern "C" size_t tgs_render_state_size(int32_t n_slots, int32_t max_per_tile) {
  if (n_slots < 0 || max_per_tile < 0 || max_per_tile > kTilePixels) return 0;
  return (size_t)n_slots * (kChunks - 1) * (size_t)raster_block(false, max_per_tile) * sizeof(float4);
}

// The workgroups of a view, 0 when it has no tile to render.
static int view_grid(const RasterArgs& a, int32_t n_st) {
  return a.valid_tiles == nullptr ? a.tiles_x * a.tiles_y : n_st;
}

static int32_t fwd_args(FwdArgs& v, const RasterArgs& a, int32_t n_st, float* out, uint32_t* ncontrib,
                        uint64_t* counters, float* state, const char* who) {
  TGS_REQUIRE(out && ncontrib, "%s: null output", who);
  TGS_REQUIRE(((uintptr_t)out & 15) == 0 && ((uintptr_t)state & 15) == 0, "%s: out and state must be 16-byte aligned",
              who);
  v.a = a;
  v.out = (float4*)out;
  v.ncontrib = ncontrib;
  v.counters = (unsigned long long*)counters;
  v.state = (float4*)state;
  v.grid = view_grid(a, n_st);
  return TGS_OK;
}

// Views of one kind (dense, or sparse with the same workgroup size).
static void fwd_launch(const Batch<FwdArgs>& b, int views, int32_t max_per_tile, hipStream_t s) {
  int grid = 0;
  for (int k = 0; k < views; ++k) grid = std::max(grid, b.v[k].grid);
  if (grid == 0) return;
  if (b.v[0].a.valid_tiles == nullptr) launch_fwd<256, true>(b, views, grid, s);
  else if (max_per_tile <= 64) launch_fwd<64, false>(b, views, grid, s);
  else if (max_per_tile <= 128) launch_fwd<128, false>(b, views, grid, s);
  else launch_fwd<256, false>(b, views, grid, s);
}

static int32_t render_fwd_launch(const RasterArgs& a, int32_t n_st, int32_t max_per_tile, float* out,
                                 uint32_t* ncontrib, uint64_t* counters, float* state, hipStream_t s,
                                 const char* who) {
  Batch<FwdArgs> b{};
  if (int32_t e = fwd_args(b.v[0], a, n_st, out, ncontrib, counters, state, who)) return e;
  fwd_launch(b, 1, max_per_tile, s);
  return hip_status(who);
}

extern "C" int32_t tgs_render_fwd(const float* splat, const uint32_t* vals, const uint32_t* ranges,
                                  int32_t tiles_x, int32_t tiles_y, int32_t width, int32_t height,
                                  const int32_t* valid_tiles, const int32_t* tile_off,
                                  const uint8_t* pix, int32_t n_st, int32_t max_per_tile,
                                  const tgs_raster_params* rp, float* out, uint32_t* ncontrib,
                                  uint64_t* counters, float* state, void* stream) {
  RasterArgs a;
  if (int32_t e = make_args(splat, vals, ranges, tiles_x, tiles_y, width, height, valid_tiles,
                            tile_off, pix, n_st, max_per_tile, rp, "tgs_render_fwd", a))
    return e;
  return render_fwd_launch(a, n_st, max_per_tile, out, ncontrib, counters, state,
                           as_stream(stream), "tgs_render_fwd");
}

extern "C" int32_t tgs_render_fwd_prefix(const float* splat, const uint32_t* vals, const uint32_t* ranges,
                                         int32_t tiles_x, int32_t tiles_y, int32_t width, int32_t height,
                                         const int32_t* valid_tiles, const int32_t* tile_off, const uint8_t* pix,
                                         int32_t n_st, int32_t max_per_tile, const tgs_raster_params* rp, float* out,
                                         uint32_t* ncontrib, uint64_t* counters, float* state, int32_t* cont_slot,
                                         uint32_t* cont_list, uint32_t* cont_count, void* stream) {
  const char* who = "tgs_render_fwd_prefix";
  RasterArgs a;
  if (int32_t e = make_args(splat, vals, ranges, tiles_x, tiles_y, width, height, valid_tiles, tile_off, pix, n_st,
                            max_per_tile, rp, who, a))
    return e;
  TGS_REQUIRE(cont_slot && cont_list && cont_count, "%s: null continuation outputs", who);
  a.mode = 1;
  a.cont_slot = cont_slot;
  a.cont_list = cont_list;
  a.cont_count = cont_count;
  hipStream_t s = as_stream(stream);
  const int64_t n_t = (int64_t)tiles_x * tiles_y;
  hipLaunchKernelGGL(fill_i32_kernel, dim3((unsigned)ceil_div(n_t, 256)), dim3(256), 0, s, cont_slot, n_t, -1,
                     cont_count);
  return render_fwd_launch(a, n_st, max_per_tile, out, ncontrib, counters, state, s, who);
}

extern "C" int32_t tgs_render_fwd_cont(const float* splat, const uint32_t* vals, const uint32_t* ranges,
                                       const uint32_t* vals2, const uint32_t* ranges2, int32_t tiles_x,
                                       int32_t tiles_y, int32_t width, int32_t height, const int32_t* valid_tiles,
                                       const int32_t* tile_off, const uint8_t* pix, int32_t n_st,
                                       int32_t max_per_tile, const tgs_raster_params* rp, const uint32_t* cont_list,
                                       const uint32_t* cont_count, float* out, uint32_t* ncontrib,
                                       uint64_t* counters, float* state, void* stream) {
  const char* who = "tgs_render_fwd_cont";
  RasterArgs a;
  if (int32_t e = make_args(splat, vals, ranges, tiles_x, tiles_y, width, height, valid_tiles, tile_off, pix, n_st,
                            max_per_tile, rp, who, a))
    return e;
  if (int32_t e = set_second(a, vals2, ranges2, who)) return e;
  TGS_REQUIRE(cont_list && cont_count, "%s: null continuation list", who);
  a.mode = 2;
  a.cont_list = (uint32_t*)cont_list;
  a.cont_count = (uint32_t*)cont_count;
  return render_fwd_launch(a, n_st, max_per_tile, out, ncontrib, counters, state,
                           as_stream(stream), who);
}

static int32_t bwd_args(BwdArgs& v, const RasterArgs& a, int32_t n_st, const float* out, const uint32_t* ncontrib,
                        const float* dL_dout, float* g2d, const float* state, uint8_t* touched,
                        const DensityArgs* dens, const char* who) {
  TGS_REQUIRE(out && ncontrib && dL_dout && g2d, "%s: null pointer", who);
  TGS_REQUIRE(((uintptr_t)out & 15) == 0 && ((uintptr_t)dL_dout & 15) == 0 && ((uintptr_t)state & 15) == 0,
              "%s: out, dL_dout and state must be 16-byte aligned", who);
  v.a = a;
  v.out = (const float4*)out;
  v.ncontrib = ncontrib;
  v.dL = (const float4*)dL_dout;
  v.g2d = g2d;
  v.state = (const float4*)state;
  v.touched = touched;
  v.dens = dens != nullptr ? *dens : DensityArgs{};
  v.grid = view_grid(a, n_st);
  return TGS_OK;
}

// Views of one kind, as in fwd_launch; all with the state record or none.
template <bool kDet = false>
static void bwd_launch(const Batch<BwdArgs>& b, int views, int32_t max_per_tile, bool density, hipStream_t s) {
  int grid = 0;
  for (int k = 0; k < views; ++k) grid = std::max(grid, b.v[k].grid);
  if (grid == 0) return;
  if (b.v[0].a.valid_tiles == nullptr) launch_bwd<256, true, kDet>(b, views, grid, density, s);
  else if (max_per_tile <= 64) launch_bwd<64, false, kDet>(b, views, grid, density, s);
  else if (max_per_tile <= 128) launch_bwd<128, false, kDet>(b, views, grid, density, s);
  else launch_bwd<256, false, kDet>(b, views, grid, density, s);
}

static int32_t render_bwd_launch(const RasterArgs& a, int32_t n_st, int32_t max_per_tile, const float* out,
                                 const uint32_t* ncontrib, const float* dL_dout, float* g2d, const float* state,
                                 uint8_t* touched, const DensityArgs* dens, hipStream_t s, const char* who) {
  Batch<BwdArgs> b{};
  if (int32_t e = bwd_args(b.v[0], a, n_st, out, ncontrib, dL_dout, g2d, state, touched, dens, who)) return e;
  bwd_launch(b, 1, max_per_tile, dens != nullptr, s);
  return hip_status(who);
}

extern "C" int32_t tgs_render_bwd(const float* splat, const uint32_t* vals, const uint32_t* ranges,
                                  int32_t tiles_x, int32_t tiles_y, int32_t width, int32_t height,
                                  const int32_t* valid_tiles, const int32_t* tile_off,
                                  const uint8_t* pix, int32_t n_st, int32_t max_per_tile,
                                  const tgs_raster_params* rp, const float* out,
                                  const uint32_t* ncontrib, const float* dL_dout, float* g2d,
                                  const float* state, uint8_t* touched, void* stream) {
  RasterArgs a;
  if (int32_t e = make_args(splat, vals, ranges, tiles_x, tiles_y, width, height, valid_tiles,
                            tile_off, pix, n_st, max_per_tile, rp, "tgs_render_bwd", a))
    return e;
  return render_bwd_launch(a, n_st, max_per_tile, out, ncontrib, dL_dout, g2d, state,
                           touched, nullptr, as_stream(stream), "tgs_render_bwd");
}

extern "C" int32_t tgs_render_bwd2(const float* splat, const uint32_t* vals, const uint32_t* ranges,
                                   const uint32_t* vals2, const uint32_t* ranges2, int32_t tiles_x, int32_t tiles_y,
                                   int32_t width, int32_t height, const int32_t* valid_tiles,
                                   const int32_t* tile_off, const uint8_t* pix, int32_t n_st, int32_t max_per_tile,
                                   const tgs_raster_params* rp, const float* out, const uint32_t* ncontrib,
                                   const float* dL_dout, float* g2d, const float* state, uint8_t* touched,
                                   const float* err, int64_t n, float* stats, void* stream) {
  const char* who = "tgs_render_bwd2";
  RasterArgs a;
  if (int32_t e = make_args(splat, vals, ranges, tiles_x, tiles_y, width, height, valid_tiles, tile_off, pix, n_st,
                            max_per_tile, rp, who, a))
    return e;
  if (int32_t e = set_second(a, vals2, ranges2, who)) return e;
  DensityArgs d{err, stats, n};
  if (stats != nullptr) {
    TGS_REQUIRE(err != nullptr && n > 0 && n < (1ll << 31), "%s: density sums need err and n", who);
    TGS_REQUIRE(((uintptr_t)stats & 15) == 0, "%s: stats must be 16-byte aligned", who);
  }
  return render_bwd_launch(a, n_st, max_per_tile, out, ncontrib, dL_dout, g2d, state,
                           touched, stats != nullptr ? &d : nullptr, as_stream(stream), who);
}

extern "C" size_t tgs_render_bwd_det_workspace_size(int64_t n_pairs, int32_t max_per_tile, int32_t dense) {
  if (n_pairs < 0 || max_per_tile < 0 || max_per_tile > kTilePixels) return 0;
  (void)dense;
  return (size_t)std::max<int64_t>(n_pairs, 1) * 9 * sizeof(float);
}

extern "C" int32_t tgs_render_bwd_deterministic(const float* splat, const uint32_t* vals, const uint32_t* ranges,
                                                int32_t tiles_x, int32_t tiles_y, int32_t width, int32_t height,
                                                const int32_t* valid_tiles, const int32_t* tile_off,
                                                const uint8_t* pix, int32_t n_st, int32_t max_per_tile,
                                                const tgs_raster_params* rp, const float* out,
                                                const uint32_t* ncontrib, const float* dL_dout, float* g2d,
                                                const float* state, uint8_t* touched, const float* depth,
                                                const int32_t* rect, int64_t n, int64_t n_pairs, void* ws,
                                                size_t ws_bytes, void* stream) {
  RasterArgs a;
  if (int32_t e = make_args(splat, vals, ranges, tiles_x, tiles_y, width, height, valid_tiles,
                            tile_off, pix, n_st, max_per_tile, rp, "tgs_render_bwd_deterministic", a))
    return e;
  TGS_REQUIRE(out && ncontrib && dL_dout && g2d && depth && rect && ws, "tgs_render_bwd_deterministic: null pointer");
  TGS_REQUIRE(n >= 0 && n < (1ll << 31) && n_pairs >= 0 && n_pairs < (1ll << 32),
              "tgs_render_bwd_deterministic: n or n_pairs out of range");
  TGS_REQUIRE(((uintptr_t)out & 15) == 0 && ((uintptr_t)dL_dout & 15) == 0 && ((uintptr_t)state & 15) == 0 &&
                  ((uintptr_t)rect & 15) == 0 && ((uintptr_t)ws & 15) == 0,
              "tgs_render_bwd_deterministic: out, dL_dout, state, rect and ws must be 16-byte aligned");
  const bool dense = valid_tiles == nullptr;
  const size_t need = tgs_render_bwd_det_workspace_size(n_pairs, max_per_tile, dense);
  TGS_REQUIRE(ws_bytes >= need, "tgs_render_bwd_deterministic: workspace %zu bytes < %zu", ws_bytes, need);
  hipStream_t s = as_stream(stream);
  float* partial = (float*)ws;
  const int64_t words = std::max<int64_t>(n_pairs, 1) * 9;
  hipLaunchKernelGGL(zero_f32_kernel, dim3((unsigned)std::min<int64_t>(ceil_div(words, 256), 8192)), dim3(256), 0,
                     s, partial, words);
  Batch<BwdArgs> b{};
  if (int32_t e = bwd_args(b.v[0], a, n_st, out, ncontrib, dL_dout, partial, state, touched, nullptr,
                           "tgs_render_bwd_deterministic"))
    return e;
  bwd_launch<true>(b, 1, max_per_tile, false, s);
  if (n > 0)
    hipLaunchKernelGGL(det_reduce_kernel, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, s, (const int4*)rect,
                       depth, vals, (const uint2*)ranges, n, tiles_x, tiles_y, partial, g2d);
  return hip_status("tgs_render_bwd_deterministic");
}

extern "C" int32_t tgs_render_bwd_density(const float* splat, const uint32_t* vals, const uint32_t* ranges,
                                          int32_t tiles_x, int32_t tiles_y, int32_t width, int32_t height,
                                          const int32_t* valid_tiles, const int32_t* tile_off,
                                          const uint8_t* pix, int32_t n_st, int32_t max_per_tile,
                                          const tgs_raster_params* rp, const float* out,
                                          const uint32_t* ncontrib, const float* dL_dout, float* g2d,
                                          const float* state, uint8_t* touched, const float* err, int64_t n,
                                          float* stats, void* stream) {
  RasterArgs a;
  if (int32_t e = make_args(splat, vals, ranges, tiles_x, tiles_y, width, height, valid_tiles,
                            tile_off, pix, n_st, max_per_tile, rp, "tgs_render_bwd_density", a))
    return e;
  TGS_REQUIRE(out && ncontrib && dL_dout && g2d && err && stats, "tgs_render_bwd_density: null pointer");
  TGS_REQUIRE(n > 0 && n < (1ll << 31), "tgs_render_bwd_density: n out of range");
  TGS_REQUIRE(((uintptr_t)stats & 15) == 0, "tgs_render_bwd_density: stats must be 16-byte aligned");
  TGS_REQUIRE(((uintptr_t)out & 15) == 0 && ((uintptr_t)dL_dout & 15) == 0 && ((uintptr_t)state & 15) == 0,
              "tgs_render_bwd_density: out, dL_dout and state must be 16-byte aligned");
  hipStream_t s = as_stream(stream);
  const DensityArgs d{err, stats, n};
  Batch<BwdArgs> b{};
  if (int32_t e = bwd_args(b.v[0], a, n_st, out, ncontrib, dL_dout, g2d, state, touched, &d, "tgs_render_bwd_density"))
    return e;
  bwd_launch(b, 1, max_per_tile, true, s);
  return hip_status("tgs_render_bwd_density");
}

static int32_t density_accumulate_launch(const RasterArgs& a, const int32_t* valid_tiles, int32_t n_st,
                                         int32_t max_per_tile, const uint32_t* ncontrib, const float* err,
                                         const float* state, int64_t n, float* stats, void* stream);

extern "C" int32_t tgs_density_accumulate(const float* splat, const uint32_t* vals, const uint32_t* ranges,
                                          int32_t tiles_x, int32_t tiles_y, int32_t width, int32_t height,
                                          const int32_t* valid_tiles, const int32_t* tile_off,
                                          const uint8_t* pix, int32_t n_st, int32_t max_per_tile,
                                          const tgs_raster_params* rp, const uint32_t* ncontrib,
                                          const float* err, const float* state, int64_t n, float* stats,
                                          void* stream) {
  RasterArgs a;
  if (int32_t e = make_args(splat, vals, ranges, tiles_x, tiles_y, width, height, valid_tiles,
                            tile_off, pix, n_st, max_per_tile, rp, "tgs_density_accumulate", a))
    return e;
  return density_accumulate_launch(a, valid_tiles, n_st, max_per_tile, ncontrib, err, state, n, stats, stream);
}

extern "C" int32_t tgs_density_accumulate2(const float* splat, const uint32_t* vals, const uint32_t* ranges,
                                           const uint32_t* vals2, const uint32_t* ranges2, int32_t tiles_x,
                                           int32_t tiles_y, int32_t width, int32_t height,
                                           const int32_t* valid_tiles, const int32_t* tile_off, const uint8_t* pix,
                                           int32_t n_st, int32_t max_per_tile, const tgs_raster_params* rp,
                                           const uint32_t* ncontrib, const float* err, const float* state,
                                           int64_t n, float* stats, void* stream) {
  RasterArgs a;
  if (int32_t e = make_args(splat, vals, ranges, tiles_x, tiles_y, width, height, valid_tiles,
                            tile_off, pix, n_st, max_per_tile, rp, "tgs_density_accumulate2", a))
    return e;
  if (int32_t e = set_second(a, vals2, ranges2, "tgs_density_accumulate2")) return e;
  return density_accumulate_launch(a, valid_tiles, n_st, max_per_tile, ncontrib, err, state, n, stats, stream);
}

static int32_t density_accumulate_launch(const RasterArgs& a, const int32_t* valid_tiles, int32_t n_st,
                                         int32_t max_per_tile, const uint32_t* ncontrib, const float* err,
                                         const float* state, int64_t n, float* stats, void* stream) {
  const int tiles_x = a.tiles_x, tiles_y = a.tiles_y;
  TGS_REQUIRE(n >= 0 && n < (1ll << 31), "tgs_density_accumulate: n out of range");
  TGS_REQUIRE(ncontrib && err && stats, "tgs_density_accumulate: null pointer");
  TGS_REQUIRE(((uintptr_t)stats & 15) == 0, "tgs_density_accumulate: stats must be 16-byte aligned");
  TGS_REQUIRE(((uintptr_t)state & 15) == 0, "tgs_density_accumulate: state must be 16-byte aligned");
  hipStream_t s = as_stream(stream);
  if (n == 0) return hip_status("tgs_density_accumulate");
  const unsigned chunks = state != nullptr ? kChunks : 1;
  const float4* st = (const float4*)state;
#define TGS_ACCUM(BLK, DENSE, GRID) \
  hipLaunchKernelGGL((render_accum_kernel<BLK, DENSE>), dim3(GRID, chunks), dim3(BLK), 0, s, a, ncontrib, err, n, \
                     stats, st)
  if (valid_tiles == nullptr) {
    TGS_ACCUM(256, true, tiles_x * tiles_y);
  } else if (n_st > 0) {
    if (max_per_tile <= 64) TGS_ACCUM(64, false, n_st);
    else if (max_per_tile <= 128) TGS_ACCUM(128, false, n_st);
    else TGS_ACCUM(256, false, n_st);
  }
#undef TGS_ACCUM
  return hip_status("tgs_density_accumulate");
}

// ------------------------------------------------------------------ several views
// A view's raster arguments; its kind decides which views share a launch.
static int32_t view_args(const tgs_view& v, const tgs_raster_params* rp, const char* who, RasterArgs& a) {
  return make_args(v.splat, v.vals, v.ranges, v.tiles_x, v.tiles_y, v.width, v.height, v.valid_tiles, v.tile_off,
                   v.pix, v.n_st, v.max_per_tile, rp, who, a);
}

static bool same_kind(const tgs_view& a, const tgs_view& b) {
  const bool dense = a.valid_tiles == nullptr;
  return dense == (b.valid_tiles == nullptr) && (a.state == nullptr) == (b.state == nullptr) &&
         raster_block(dense, a.max_per_tile) == raster_block(dense, b.max_per_tile);
}

// Views [k, end) that share a launch.
static int32_t kind_end(const tgs_view* views, int32_t n_views, int32_t k) {
  int32_t end = k + 1;
  while (end < n_views && end - k < kBatch && same_kind(views[k], views[end])) ++end;
  return end;
}

extern "C" int32_t tgs_render_fwd_views(const tgs_view* views, int32_t n_views, const tgs_raster_params* rp,
                                        uint64_t* counters, void* stream) {
  const char* who = "tgs_render_fwd_views";
  TGS_REQUIRE(n_views >= 0 && (n_views == 0 || views != nullptr), "%s: bad view list", who);
  for (int pass = 0; pass < 2; ++pass)  // every view is checked before any is launched
    for (int32_t k = 0, end; k < n_views; k = end) {
      end = kind_end(views, n_views, k);
      Batch<FwdArgs> b{};
      for (int32_t i = k; i < end; ++i) {
        RasterArgs a;
        if (int32_t e = view_args(views[i], rp, who, a)) return e;
        if (int32_t e = fwd_args(b.v[i - k], a, views[i].n_st, views[i].out, views[i].ncontrib, counters,
                                 views[i].state, who))
          return e;
      }
      if (pass == 1) fwd_launch(b, end - k, views[k].max_per_tile, as_stream(stream));
    }
  return hip_status(who);
}

extern "C" int32_t tgs_render_bwd_views(const tgs_view* views, int32_t n_views, const tgs_raster_params* rp,
                                        uint8_t* touched, int64_t n, float* stats, void* stream) {
  const char* who = "tgs_render_bwd_views";
  TGS_REQUIRE(n_views >= 0 && (n_views == 0 || views != nullptr), "%s: bad view list", who);
  if (stats != nullptr) {
    TGS_REQUIRE(n > 0 && n < (1ll << 31), "%s: n out of range", who);
    TGS_REQUIRE(((uintptr_t)stats & 15) == 0, "%s: stats must be 16-byte aligned", who);
  }
  for (int pass = 0; pass < 2; ++pass)
    for (int32_t k = 0, end; k < n_views; k = end) {
      end = kind_end(views, n_views, k);
      Batch<BwdArgs> b{};
      for (int32_t i = k; i < end; ++i) {
        const tgs_view& v = views[i];
        RasterArgs a;
        if (int32_t e = view_args(v, rp, who, a)) return e;
        TGS_REQUIRE(stats == nullptr || v.err != nullptr, "%s: density sums need err", who);
        const DensityArgs d{v.err, stats, n};
        if (int32_t e = bwd_args(b.v[i - k], a, v.n_st, v.out, v.ncontrib, v.dL_dout, v.g2d, v.state, touched,
                                 stats != nullptr ? &d : nullptr, who))
          return e;
      }
      if (pass == 1) bwd_launch(b, end - k, views[k].max_per_tile, stats != nullptr, as_stream(stream));
    }
  return hip_status(who);
}
