// Sparse supervision (Charbonnier L1 + tile NCC with gradient balance, or the
// tile S-SSIM of the ablation in its place) and the per-pixel error/age maps.
//
// loss: one wave per sampled tile; a lane holds up to four of the tile's
// samples (strided, so loads coalesce).  The tile statistics (means, centred
// second moments, NCC per channel, the two mean gradient norms) are wave
// sums through DPP; everything stays in registers between the passes.
// ema_age: one workgroup per band of eight tiles of a tile row; the sample
// lists are scattered into an LDS slot table and each thread updates eight
// consecutive pixels of a row (16-byte age-map accesses).
#include <hip/hip_fp16.h>

#include "common.h"

namespace tgs {

// SSIM constants for values in [0, 1]: (0.01)^2 and (0.03)^2.
constexpr float kSsimC1 = 1e-4f;
constexpr float kSsimC2 = 9e-4f;

// A view's arguments; the views of a step share a launch, one per grid layer.
struct LossArgs {
  const float4* out;
  const float* gt;
  const int32_t* valid_tiles;
  const int32_t* tile_off;
  const uint8_t* pix;
  float4* dL;
  float* err;
  float* lambda_out;
  float2* tile_loss;
  int H, W, tiles_x;
  int grid;  // the view's workgroups; the launch's grid is the largest view's
};

template <bool kDense, bool kSsim = false>
__global__ void __launch_bounds__(64) loss_kernel(Batch<LossArgs> batch, const int64_t* __restrict__ totals,
                                                  float eps_c2, float eps_n, float eps_l) {
  const LossArgs& v = batch.v[blockIdx.z];
  if ((int)blockIdx.x >= v.grid) return;
  const float4* __restrict__ const out = v.out;
  const float* __restrict__ const gt = v.gt;
  const int32_t* __restrict__ const valid_tiles = v.valid_tiles;
  const int32_t* __restrict__ const tile_off = v.tile_off;
  const uint8_t* __restrict__ const pix = v.pix;
  float4* __restrict__ const dL = v.dL;
  float* __restrict__ const err = v.err;
  float* __restrict__ const lambda_out = v.lambda_out;
  float2* __restrict__ const tile_loss = v.tile_loss;
  const int H = v.H, W = v.W, tiles_x = v.tiles_x;
  const int slot = blockIdx.x, lane = threadIdx.x;
  const int tile = kDense ? slot : valid_tiles[slot];
  const int tx = tile % tiles_x, ty = tile / tiles_x;
  const int p0 = kDense ? 0 : tile_off[slot];
  const int np = kDense ? kTilePixels : tile_off[slot + 1] - p0;
  const int64_t HW = (int64_t)H * W;

  bool in[4];
  int64_t oi[4];
  float x[4][3], y[4][3];
  float s[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  int cnt = 0;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int k = lane + 64 * r;
    int loc = -1;
    if (kDense) {
      loc = k;
    } else if (k < np) {
      loc = pix[p0 + k];
    }
    const int px = tx * kTile + (loc & 15), py = ty * kTile + (loc >> 4);
    in[r] = loc >= 0 && px < W && py < H;
    oi[r] = kDense ? (int64_t)py * W + px : (int64_t)p0 + k;
    if (in[r]) {
      const float4 o = out[oi[r]];
      const int64_t gi = (int64_t)py * W + px;
      x[r][0] = o.x; x[r][1] = o.y; x[r][2] = o.z;
      y[r][0] = gt[gi]; y[r][1] = gt[HW + gi]; y[r][2] = gt[2 * HW + gi];
      for (int c = 0; c < 3; ++c) {
        s[c] += x[r][c];
        s[3 + c] += y[r][c];
      }
      ++cnt;
    } else {
      for (int c = 0; c < 3; ++c) x[r][c] = y[r][c] = 0.f;
    }
  }
  const float n = (float)wave_sum_i(cnt);
  if (n == 0.f) return;
  const float inv_n = 1.f / n;
  float mx[3], my[3];
  for (int c = 0; c < 3; ++c) {
    mx[c] = wave_sum(s[c]) * inv_n;
    my[c] = wave_sum(s[3 + c]) * inv_n;
  }
  float m2[9] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};  // Vx, Vy, Cxy per channel
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if (!in[r]) continue;
    for (int c = 0; c < 3; ++c) {
      const float xc = x[r][c] - mx[c], yc = y[r][c] - my[c];
      m2[c] += xc * xc;
      m2[3 + c] += yc * yc;
      m2[6 + c] += xc * yc;
    }
  }
  // structure term per channel: NCC, or SSIM (ncc[] then holds SSIM and the
  // per-sample gradient below uses the SSIM factors A1, A2, B1, B2)
  float Vy[3], D[3], rsD[3], ncc[3], A1[3], A2[3], B1[3], B2[3];
  for (int c = 0; c < 3; ++c) {
    const float Vx = wave_sum(m2[c]) * inv_n;
    Vy[c] = wave_sum(m2[3 + c]) * inv_n;
    const float Cxy = wave_sum(m2[6 + c]) * inv_n;
    if constexpr (kSsim) {
      A1[c] = 2.f * mx[c] * my[c] + kSsimC1;
      A2[c] = 2.f * Cxy + kSsimC2;
      B1[c] = mx[c] * mx[c] + my[c] * my[c] + kSsimC1;
      B2[c] = Vx + Vy[c] + kSsimC2;
      ncc[c] = (A1[c] * A2[c]) / (B1[c] * B2[c]);
    } else {
      D[c] = Vx * Vy[c] + eps_n;
      rsD[c] = 1.f / sqrtf(D[c]);
      ncc[c] = Cxy * rsD[c];
    }
  }
  // per-sample gradients and their mean L1 norms
  float g1[4][3], gn[4][3];
  float n1 = 0.f, nn = 0.f, rho_sum = 0.f;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    for (int c = 0; c < 3; ++c) {
      g1[r][c] = 0.f;
      gn[r][c] = 0.f;
    }
    if (!in[r]) continue;
    for (int c = 0; c < 3; ++c) {
      const float d = x[r][c] - y[r][c];
      const float rho = sqrtf(d * d + eps_c2);
      rho_sum += rho;
      g1[r][c] = d / rho;
      const float xc = x[r][c] - mx[c], yc = y[r][c] - my[c];
      if constexpr (kSsim)
        gn[r][c] = -2.f * ncc[c] * (my[c] / A1[c] + yc / A2[c] - mx[c] / B1[c] - xc / B2[c]);
      else
        gn[r][c] = -(yc * rsD[c] - ncc[c] * Vy[c] * xc / D[c]);
      n1 += fabsf(g1[r][c]);
      nn += fabsf(gn[r][c]);
    }
  }
  const float gbar1 = wave_sum(n1) * inv_n, gbarn = wave_sum(nn) * inv_n;
  const float lam = fminf(fmaxf(gbar1 / (gbarn + eps_l), 0.f), 1.f);
  const float P_step = (float)totals[0], T_step = (float)totals[1];
  const float k1 = 1.f / (3.f * P_step), kn = lam / (3.f * n * T_step);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if (!in[r]) continue;
    dL[oi[r]] = make_float4(g1[r][0] * k1 + gn[r][0] * kn, g1[r][1] * k1 + gn[r][1] * kn,
                            g1[r][2] * k1 + gn[r][2] * kn, 0.f);
    err[oi[r]] = fabsf(x[r][0] - y[r][0]) + fabsf(x[r][1] - y[r][1]) + fabsf(x[r][2] - y[r][2]);
  }
  const float rho_tot = wave_sum(rho_sum);
  if (lane == 0) {
    lambda_out[slot] = lam;
    tile_loss[slot] = make_float2(rho_tot * k1, lam * (1.f - (ncc[0] + ncc[1] + ncc[2]) / 3.f) / T_step);
  }
}

__device__ __forceinline__ uint16_t ema_half(uint16_t e_bits, float e, float beta, float omb) {
#pragma clang fp contract(off)
  const float E = __half2float(__ushort_as_half(e_bits));
  const float t1 = omb * E;
  const float t2 = beta * e;
  return __half_as_ushort(__float2half_rn(t1 + t2));
}

// One workgroup per band of kEmaTiles tiles of a tile row (16 rows x 128
// pixels); a thread takes 8 consecutive pixels of one row, so the age map
// moves in 16-byte accesses.  The band's sample lists are first scattered
// into LDS (for each pixel: its sample index or -1); a sampled pixel gets
// age 0 and its error blended, every other pixel age + 1 (saturating).
constexpr int kEmaTiles = 8;

struct EmaArgs {
  uint16_t* E;
  uint16_t* A;
  const int32_t* tile_slot;
  const int32_t* tile_off;
  const uint8_t* pix;
  const float* err;
  int H, W, tiles_x, tiles_y;
};

__global__ void __launch_bounds__(256) ema_age_kernel(Batch<EmaArgs> batch, float beta, float omb) {
  const EmaArgs& v = batch.v[blockIdx.z];
  if ((int)blockIdx.x * kEmaTiles >= v.tiles_x || (int)blockIdx.y >= v.tiles_y) return;
  uint16_t* __restrict__ const E = v.E;
  uint16_t* __restrict__ const A = v.A;
  const int32_t* __restrict__ const tile_slot = v.tile_slot;
  const int32_t* __restrict__ const tile_off = v.tile_off;
  const uint8_t* __restrict__ const pix = v.pix;
  const float* __restrict__ const err = v.err;
  const int H = v.H, W = v.W, tiles_x = v.tiles_x;
  __shared__ int pos[kEmaTiles][kTilePixels];
  const int tid = threadIdx.x, ty = blockIdx.y, tx0 = blockIdx.x * kEmaTiles;
  for (int k = 0; k < kEmaTiles; ++k) pos[k][tid] = -1;
  __syncthreads();
  for (int k = 0; k < kEmaTiles; ++k) {
    const int tx = tx0 + k;
    if (tx >= tiles_x) break;
    const int slot = tile_slot[ty * tiles_x + tx];
    if (slot >= 0) {
      const int p0 = tile_off[slot], np = tile_off[slot + 1] - p0;
      if (tid < np) pos[k][pix[p0 + tid]] = p0 + tid;
    }
  }
  __syncthreads();
  const int row = tid >> 4, seg = tid & 15;  // 16 rows x 16 segments of 8 pixels
  const int y = ty * kTile + row, x0 = tx0 * kTile + seg * 8;
  if (y >= H || x0 >= W) return;
  const int k = seg >> 1, lx0 = (seg & 1) * 8;  // tile of the band, first local column
  const int64_t i0 = (int64_t)y * W + x0;
  uint16_t a[8];
  const bool vec = (W & 7) == 0 && x0 + 8 <= W;  // 16-byte aligned and inside the row
  if (vec) {
    const uint4 q = *reinterpret_cast<const uint4*>(A + i0);
    const uint32_t w[4] = {q.x, q.y, q.z, q.w};
    for (int j = 0; j < 4; ++j) {
      a[2 * j] = (uint16_t)(w[j] & 0xffffu);
      a[2 * j + 1] = (uint16_t)(w[j] >> 16);
    }
  } else {
    for (int j = 0; j < 8; ++j) a[j] = x0 + j < W ? A[i0 + j] : 0;
  }
  for (int j = 0; j < 8; ++j) {
    const int p = pos[k][row * kTile + lx0 + j];
    if (p >= 0) {
      a[j] = 0;
      E[i0 + j] = ema_half(E[i0 + j], err[p], beta, omb);
    } else {
      a[j] = a[j] == 0xffffu ? a[j] : (uint16_t)(a[j] + 1u);
    }
  }
  if (vec) {
    uint4 q;
    q.x = (uint32_t)a[0] | ((uint32_t)a[1] << 16);
    q.y = (uint32_t)a[2] | ((uint32_t)a[3] << 16);
    q.z = (uint32_t)a[4] | ((uint32_t)a[5] << 16);
    q.w = (uint32_t)a[6] | ((uint32_t)a[7] << 16);
    *reinterpret_cast<uint4*>(A + i0) = q;
  } else {
    for (int j = 0; j < 8; ++j)
      if (x0 + j < W) A[i0 + j] = a[j];
  }
}

__global__ void __launch_bounds__(256) error_init_kernel(const float4* __restrict__ out,
                                                         const float* __restrict__ gt, int64_t HW,
                                                         uint16_t* __restrict__ E) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= HW) return;
  const float4 o = out[i];
  float e;
  {
#pragma clang fp contract(off)
    e = (fabsf(o.x - gt[i]) + fabsf(o.y - gt[HW + i])) + fabsf(o.z - gt[2 * HW + i]);
  }
  E[i] = __half_as_ushort(__float2half_rn(e));
}

}  // namespace tgs

using namespace tgs;

static int32_t loss_params_check(const tgs_loss_params* lp, const int64_t* totals, const char* who) {
  TGS_REQUIRE(lp != nullptr, "%s: null params", who);
  TGS_REQUIRE(totals != nullptr, "%s: null pointer", who);
  TGS_REQUIRE(lp->structure == TGS_STRUCTURE_NCC || lp->structure == TGS_STRUCTURE_SSIM,
              "%s: unknown structure term %d", who, lp->structure);
  return TGS_OK;
}

static int32_t loss_args(LossArgs& v, const float* out, const float* gt, int32_t height, int32_t width,
                         const int32_t* valid_tiles, const int32_t* tile_off, const uint8_t* pix, int32_t n_st,
                         float* dL_dout, float* err, float* lambda, float* tile_loss, const char* who) {
  TGS_REQUIRE(height > 0 && width > 0, "%s: bad image size", who);
  TGS_REQUIRE(out && gt && dL_dout && err && lambda && tile_loss, "%s: null pointer", who);
  TGS_REQUIRE(((uintptr_t)out & 15) == 0 && ((uintptr_t)dL_dout & 15) == 0,
              "%s: out and dL_dout must be 16-byte aligned", who);
  const int tiles_x = (int)ceil_div(width, kTile), tiles_y = (int)ceil_div(height, kTile);
  if (valid_tiles != nullptr) {
    TGS_REQUIRE(tile_off && pix, "%s: null tile_off/pix", who);
    TGS_REQUIRE(n_st >= 0 && n_st <= tiles_x * tiles_y, "%s: bad n_st %d", who, n_st);
  }
  v = LossArgs{(const float4*)out, gt, valid_tiles, tile_off, pix, (float4*)dL_dout, err, lambda, (float2*)tile_loss,
               height, width, tiles_x, valid_tiles == nullptr ? tiles_x * tiles_y : n_st};
  return TGS_OK;
}

// Views that are all dense or all sparse.
static void loss_launch(const Batch<LossArgs>& b, int views, const int64_t* totals, const tgs_loss_params* lp,
                        hipStream_t s) {
  int grid = 0;
  for (int k = 0; k < views; ++k) grid = max(grid, b.v[k].grid);
  if (grid == 0) return;
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)grid, 1, (unsigned)views), dim3(64), 0, s, b, totals,
                       lp->eps_charb * lp->eps_charb, lp->eps_ncc, lp->eps_lambda);
  };
  const bool ssim = lp->structure == TGS_STRUCTURE_SSIM;
  if (b.v[0].valid_tiles == nullptr) {
    if (ssim) launch(loss_kernel<true, true>);
    else launch(loss_kernel<true, false>);
  } else {
    if (ssim) launch(loss_kernel<false, true>);
    else launch(loss_kernel<false, false>);
  }
}

extern "C" int32_t tgs_loss(const float* out, const float* gt, int32_t height, int32_t width,
                            const int32_t* valid_tiles, const int32_t* tile_off, const uint8_t* pix,
                            int32_t n_st, const int64_t* totals, const tgs_loss_params* lp,
                            float* dL_dout, float* err, float* lambda, float* tile_loss,
                            void* stream) {
  if (int32_t e = loss_params_check(lp, totals, "tgs_loss")) return e;
  Batch<LossArgs> b{};
  if (int32_t e = loss_args(b.v[0], out, gt, height, width, valid_tiles, tile_off, pix, n_st, dL_dout, err, lambda,
                            tile_loss, "tgs_loss"))
    return e;
  loss_launch(b, 1, totals, lp, as_stream(stream));
  return hip_status("tgs_loss");
}

extern "C" int32_t tgs_loss_views(const tgs_view* views, int32_t n_views, const int64_t* totals,
                                  const tgs_loss_params* lp, void* stream) {
  const char* who = "tgs_loss_views";
  TGS_REQUIRE(n_views >= 0 && (n_views == 0 || views != nullptr), "%s: bad view list", who);
  if (int32_t e = loss_params_check(lp, totals, who)) return e;
  for (int pass = 0; pass < 2; ++pass)  // every view is checked before any is launched
    for (int32_t k = 0, end; k < n_views; k = end) {
      Batch<LossArgs> b{};
      for (end = k; end < n_views && end - k < kBatch; ++end) {
        const tgs_view& v = views[end];
        if ((v.valid_tiles == nullptr) != (views[k].valid_tiles == nullptr)) break;
        if (int32_t e = loss_args(b.v[end - k], v.out, v.gt, v.height, v.width, v.valid_tiles, v.tile_off, v.pix,
                                  v.n_st, v.dL_dout, v.err, v.lambda, v.tile_loss, who))
          return e;
      }
      if (pass == 1) loss_launch(b, end - k, totals, lp, as_stream(stream));
    }
  return hip_status(who);
}

static int32_t ema_args(EmaArgs& v, uint16_t* E, uint16_t* A, int32_t height, int32_t width, const int32_t* tile_slot,
                        const int32_t* tile_off, const uint8_t* pix, const float* err, const char* who) {
  TGS_REQUIRE(height > 0 && width > 0, "%s: bad image size", who);
  TGS_REQUIRE(E && A && tile_slot && tile_off && pix && err, "%s: null pointer", who);
  TGS_REQUIRE((width & 7) != 0 || ((uintptr_t)A & 15) == 0,
              "%s: A must be 16-byte aligned when the width is a multiple of 8", who);
  v = EmaArgs{E,   A,      tile_slot, tile_off, pix, err, height, width, (int)ceil_div(width, kTile),
              (int)ceil_div(height, kTile)};
  return TGS_OK;
}

static void ema_launch(const Batch<EmaArgs>& b, int views, float beta, hipStream_t s) {
  int tx = 0, ty = 0;
  for (int k = 0; k < views; ++k) {
    tx = max(tx, b.v[k].tiles_x);
    ty = max(ty, b.v[k].tiles_y);
  }
  hipLaunchKernelGGL(ema_age_kernel, dim3((unsigned)ceil_div(tx, kEmaTiles), (unsigned)ty, (unsigned)views), dim3(256),
                     0, s, b, beta, 1.0f - beta);
}

extern "C" int32_t tgs_ema_age_update(uint16_t* E, uint16_t* A, int32_t height, int32_t width,
                                      const int32_t* tile_slot, const int32_t* tile_off,
                                      const uint8_t* pix, const float* err, float beta,
                                      void* stream) {
  Batch<EmaArgs> b{};
  if (int32_t e = ema_args(b.v[0], E, A, height, width, tile_slot, tile_off, pix, err, "tgs_ema_age_update")) return e;
  ema_launch(b, 1, beta, as_stream(stream));
  return hip_status("tgs_ema_age_update");
}

extern "C" int32_t tgs_ema_age_update_views(const tgs_view* views, int32_t n_views, float beta, void* stream) {
  const char* who = "tgs_ema_age_update_views";
  TGS_REQUIRE(n_views >= 0 && (n_views == 0 || views != nullptr), "%s: bad view list", who);
  for (int32_t i = 0; i < n_views; ++i)
    for (int32_t j = 0; j < i; ++j)
      TGS_REQUIRE(views[i].E != views[j].E && views[i].A != views[j].A, "%s: views %d and %d share a map", who, j, i);
  for (int pass = 0; pass < 2; ++pass)
    for (int32_t k = 0; k < n_views; k += kBatch) {
      const int nv = min(kBatch, n_views - k);
      Batch<EmaArgs> b{};
      for (int i = 0; i < nv; ++i) {
        const tgs_view& v = views[k + i];
        if (int32_t e = ema_args(b.v[i], v.E, v.A, v.height, v.width, v.tile_slot, v.tile_off, v.pix, v.err, who))
          return e;
      }
      if (pass == 1) ema_launch(b, nv, beta, as_stream(stream));
    }
  return hip_status(who);
}

extern "C" int32_t tgs_error_init(const float* out_dense, const float* gt, int32_t height,
                                  int32_t width, uint16_t* E, void* stream) {
  TGS_REQUIRE(height > 0 && width > 0, "tgs_error_init: bad image size");
  TGS_REQUIRE(out_dense && gt && E, "tgs_error_init: null pointer");
  const int64_t HW = (int64_t)height * width;
  hipLaunchKernelGGL(error_init_kernel, dim3((unsigned)ceil_div(HW, 256)), dim3(256), 0,
                     as_stream(stream), (const float4*)out_dense, gt, HW, E);
  return hip_status("tgs_error_init");
}
