// EWA projection with SH colour (forward) and its chain rule (backward).
//
// One thread per Gaussian, FP64 arithmetic.  Both kernels are HBM-bound
// (59 floats in, 12-17 out per Gaussian), so FP64 costs nothing measurable
// on gfx950 (78.6 TFLOP/s FP64) and keeps the integer decisions (depth key
// bits, tile rectangle, radius) identical to an FP64 reference written in
// the same operation order.  Parameters are read row by row from the
// [59][n] store, so every load is coalesced across the wave.
#include <algorithm>

#include "projection.h"

// The depth, centre and rectangle must follow a fixed sequence of rounded
// operations; no multiply-add contraction in this file.
#pragma clang fp contract(off)

namespace tgs {

// The outputs of one view, and its camera.
struct ProjectView {
  CamArgs cam;
  float4* splat;
  float* depth;
  int* radius;
  int4* rect;
  uint8_t* clampm;
  float* g2d_clear;
};

// Views of one launch: a step's views share the read of the parameters (236
// bytes per Gaussian, against 109 written per view), which bounds the kernel:
// three views of 1.5M Gaussians take 201 us in one launch, 3 x 116 us in three.
// The records are kernel arguments, at most 4 KB.
constexpr int kProjectViews = 8;
struct ProjectViews {
  ProjectView v[kProjectViews];
};

// PT = float: the training path.  PT = double: the FP64 instantiation for
// gradient checks, which also writes the splat record in doubles (rec64:
// centre x, y; conic a, b, c; opacity; r, g, b; depth; two zeros).
// The splat records (48 bytes per Gaussian) and the cleared gradient
// records (36 bytes) of a wave's 64 Gaussians are contiguous, so they are
// written as whole runs: the splat floats staged in LDS, then every lane
// storing consecutive 16-byte pieces (and 4-byte zeros for the gradient),
// instead of each lane writing its own records at a 48- or 36-byte stride.
template <typename PT, int kDeg, bool kMulti>
__global__ void __launch_bounds__(256, kMulti ? 4 : 1) project_fwd_kernel(const PT* __restrict__ params, int64_t n, int n_views,
                                                          ProjectViews views, double z_near, double dil,
                                                          double* __restrict__ rec64) {
  __shared__ float4 s_rec[256 / kWave][3 * kWave];
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool valid = i < n;
  const int64_t ic = valid ? i : n - 1;  // lanes past the end compute on a valid Gaussian and store nothing
  const int lane = lane_id(), wave = (int)threadIdx.x / kWave;
  const int64_t w0 = i - lane;  // the wave's first Gaussian
  if (w0 >= n) return;          // wave-uniform; nothing below waits for the workgroup
  // the SH coefficients are loaded with the geometry rows, before anything
  // depends on them (one round trip to memory; culled Gaussians read them
  // for nothing, a small share of the traffic)
  constexpr int nk = (kDeg + 1) * (kDeg + 1);
  PT cf[3 * nk];
#pragma unroll
  for (int q = 0; q < 3 * nk; ++q) cf[q] = params[(int64_t)(11 + q) * n + ic];
  Geom g;
  shape_geometry(params, n, ic, g);
  const double opac = 1.0 / (1.0 + exp(-(double)params[10 * n + ic]));
  float4* const sr = s_rec[wave];
#pragma unroll 1
  for (int q = 0; q < (kMulti ? n_views : 1); ++q) {
    const ProjectView& view = views.v[q];
    const CamArgs& cam = view.cam;
    // the coefficients stay as loaded: widened outside the loop they would
    // take twice the registers over all views
    if constexpr (kMulti) {
#pragma unroll
      for (int k = 0; k < 3 * nk; ++k) asm volatile("" : "+v"(cf[k]));
    }
    if (view.g2d_clear != nullptr) {
      const int64_t end = n * TGS_G2D_FLOATS;
#pragma unroll
      for (int k = 0; k < TGS_G2D_FLOATS; ++k) {
        const int64_t e = w0 * TGS_G2D_FLOATS + k * kWave + lane;
        if (e < end) view.g2d_clear[e] = 0.f;
      }
    }
    view_geometry(cam, z_near, dil, g);
    float4 r0 = make_float4(0.f, 0.f, 0.f, 0.f), r1 = r0, r2 = make_float4(0.f, 0.f, 0.f, (float)g.t[2]);
    int rad = 0;
    int4 rc = make_int4(0, 0, 0, 0);
    uint8_t cm = 0;
    if (g.visible) {
      // view-dependent colour
      const double dx = g.mu[0] - cam.center[0], dy = g.mu[1] - cam.center[1],
                   dz = g.mu[2] - cam.center[2];
      const double dn = sqrt(dx * dx + dy * dy + dz * dz);
      const double ux = dx / dn, uy = dy / dn, uz = dz / dn;
      double rgb[3] = {0.5, 0.5, 0.5};
#pragma unroll
      for (int k = 0; k < nk; ++k) {
        double Yk, g0, g1, g2;
        sh_term(k, ux, uy, uz, Yk, g0, g1, g2);
        for (int ch = 0; ch < 3; ++ch) rgb[ch] += Yk * (double)cf[3 * k + ch];
      }
      for (int ch = 0; ch < 3; ++ch)
        if (rgb[ch] < 0.0) {
          rgb[ch] = 0.0;
          cm |= (uint8_t)(1u << ch);
        }
      const double fxp = floor(g.px), fyp = floor(g.py);
      r0 = make_float4((float)fxp, (float)fyp, (float)(g.px - fxp), (float)(g.py - fyp));
      // the conic Q = Sigma'^-1 = [[c, -b], [-b, a]] / det in its LDL^T form:
      // Q_00 = c / det, beta = Q_01 / Q_00 = -b / c, delta = det Q / Q_00 = 1 / c
      r1 = make_float4((float)(g.c / g.det), (float)(-g.b / g.c), (float)(1.0 / g.c), (float)opac);
      r2 = make_float4((float)rgb[0], (float)rgb[1], (float)rgb[2], (float)g.t[2]);
      rad = (int)g.radius;
      rc = make_int4(g.rect[0], g.rect[1], g.rect[2], g.rect[3]);
      if (rec64 != nullptr && valid) {
        const double r64[12] = {g.px, g.py, g.c / g.det, -g.b / g.det, g.a / g.det, opac,
                                rgb[0], rgb[1], rgb[2], g.t[2], 0.0, 0.0};
        for (int k = 0; k < 12; ++k) rec64[12 * i + k] = r64[k];
      }
    } else if (rec64 != nullptr && valid) {
      for (int k = 0; k < 12; ++k) rec64[12 * i + k] = k == 9 ? g.t[2] : 0.0;
    }
    if (valid) {
      view.depth[i] = (float)g.t[2];
      view.radius[i] = rad;
      view.rect[i] = rc;
      view.clampm[i] = cm;
    }
    // the wave's own LDS, whose operations execute in order
    sr[3 * lane] = r0;
    sr[3 * lane + 1] = r1;
    sr[3 * lane + 2] = r2;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int64_t end = n * 3;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int64_t e = w0 * 3 + k * kWave + lane;
      if (e < end) view.splat[e] = sr[k * kWave + lane];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// accumulate: grad += gradient; otherwise grad = gradient, with zeros for
// culled Gaussians (every row of every Gaussian is written once).
//
// A workgroup takes kItems x 256 consecutive Gaussians.  Those without a
// gradient (at sparse rates most of them) only have their rows cleared, in
// whole lines; the others are listed in LDS and spread over the threads, so a
// wave's FP64 chain runs for 64 of them and not for the few among 64
// neighbours.  With few Gaussians (kItems = 1) a thread keeps its own.  300k
// Gaussians at 1296x840, a quarter of the pixels: 60 us without lists, 46 with.
template <typename PT, int kItems>
__global__ void __launch_bounds__(256) project_bwd_kernel(
    const PT* __restrict__ params, int64_t n, CamArgs cam, int sh_degree, double z_near,
    double dil, const int* __restrict__ radius, const uint8_t* __restrict__ clampm,
    const PT* __restrict__ g2d, PT* __restrict__ grad, bool accumulate) {
  // culled, or no screen-space gradient in this view: the gradient is zero, so
  // nothing is added, or zeros are written, without reading the parameters
  auto has_gradient = [&](int64_t i) {
    bool any = false;
    if (i < n && radius[i] != 0)
      for (int k = 0; k < 9; ++k) any = any || (double)g2d[i * 9 + k] != 0.0;
    if (i < n && !any && !accumulate)
      for (int r = 0; r < TGS_PARAM_ROWS; ++r) grad[(int64_t)r * n + i] = (PT)0;
    return any;
  };
  auto one = [&](int64_t i) {
    double gg[9];
    for (int k = 0; k < 9; ++k) gg[k] = (double)g2d[i * 9 + k];
    Geom g;
    geometry(params, n, i, cam, z_near, dil, g);
    chain_rule(params, n, i, cam, sh_degree, g, gg, clampm[i], [&](int row, double v) {
      const int64_t idx = (int64_t)row * n + i;
      grad[idx] = accumulate ? grad[idx] + (PT)v : (PT)v;
    });
  };
  const int64_t w0 = (int64_t)blockIdx.x * (256 * kItems);
  if constexpr (kItems == 1) {
    if (has_gradient(w0 + threadIdx.x)) one(w0 + threadIdx.x);
  } else {
    __shared__ uint16_t s_list[256 * kItems];
    __shared__ int s_count;
    if (threadIdx.x == 0) s_count = 0;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kItems; ++q) {
      const int at = q * 256 + (int)threadIdx.x;
      const bool any = has_gradient(w0 + at);
      const uint64_t m = ballot(any);
      int base = 0;
      if (m != 0ull) {
        if (lane_id() == 0) base = atomicAdd(&s_count, __popcll(m));
        base = __builtin_amdgcn_readfirstlane(base);
      }
      if (any) s_list[base + mask_rank(m)] = (uint16_t)at;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < s_count; e += 256) one(w0 + s_list[e]);
  }
}

// The window is the largest of 256, 512 and 1024 with more than kBwdWindows
// windows (one to a compute unit).
constexpr int64_t kBwdWindows = 256;

template <typename PT>
static void launch_project_bwd(const PT* params, int64_t n, const tgs_camera* cam, const tgs_raster_params* rp,
                               const int32_t* radius, const uint8_t* clamp, const PT* g2d, PT* grad, bool accumulate,
                               hipStream_t s) {
  const CamArgs ca = make_cam(cam);
  auto launch = [&](auto kernel, int64_t window) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)ceil_div(n, window)), dim3(256), 0, s, params, n, ca, rp->sh_degree,
                       (double)rp->z_near, (double)rp->dilation, radius, clamp, g2d, grad, accumulate);
  };
  if (n > 1024 * kBwdWindows) launch(project_bwd_kernel<PT, 4>, 1024);
  else if (n > 512 * kBwdWindows) launch(project_bwd_kernel<PT, 2>, 512);
  else launch(project_bwd_kernel<PT, 1>, 256);
}

}  // namespace tgs

using namespace tgs;


template <typename PT>
static void launch_project(const PT* params, int64_t n, int n_views, const ProjectViews& views,
                           const tgs_raster_params* rp, double* rec64, hipStream_t s) {
  const int block = 256;
  const dim3 grid((unsigned)ceil_div(n, block));
#define TGS_PROJECT(D, M)                                                                                      \
  hipLaunchKernelGGL((project_fwd_kernel<PT, D, M>), grid, dim3(block), 0, s, params, n, n_views, views,       \
                     (double)rp->z_near, (double)rp->dilation, rec64)
#define TGS_PROJECT_DEG(M)                \
  switch (rp->sh_degree) {                \
    case 0: TGS_PROJECT(0, M); break;     \
    case 1: TGS_PROJECT(1, M); break;     \
    case 2: TGS_PROJECT(2, M); break;     \
    default: TGS_PROJECT(3, M); break;    \
  }
  if constexpr (sizeof(PT) == 4) {
    if (n_views > 1) {
      TGS_PROJECT_DEG(true)
      return;
    }
  }
  TGS_PROJECT_DEG(false)
#undef TGS_PROJECT_DEG
#undef TGS_PROJECT
}

extern "C" int32_t tgs_project_views(const float* params, int64_t n, int32_t n_views, const tgs_camera* cams,
                                     const tgs_raster_params* rp, float* const* splat, float* const* depth,
                                     int32_t* const* radius, int32_t* const* rect, uint8_t* const* clamp,
                                     float* const* g2d_clear, void* stream) {
  const char* who = "tgs_project_views";
  TGS_REQUIRE(n >= 0, "%s: n < 0", who);
  TGS_REQUIRE(n_views >= 0 && (n_views == 0 || cams != nullptr), "%s: bad views", who);
  if (int32_t e = check_raster_params(rp)) return e;
  for (int k = 0; k < n_views; ++k)
    TGS_REQUIRE(cams[k].width > 0 && cams[k].height > 0, "%s: bad camera %d", who, k);
  if (n == 0 || n_views == 0) return TGS_OK;
  TGS_REQUIRE(params && splat && depth && radius && rect && clamp, "%s: null pointer", who);
  for (int k = 0; k < n_views; ++k) {
    TGS_REQUIRE(splat[k] && depth[k] && radius[k] && rect[k] && clamp[k], "%s: null output of view %d", who, k);
    TGS_REQUIRE(((uintptr_t)splat[k] & 15) == 0 && ((uintptr_t)rect[k] & 15) == 0,
                "%s: splat and rect must be 16-byte aligned", who);
  }
  for (int k0 = 0; k0 < n_views; k0 += kProjectViews) {
    ProjectViews views{};
    const int c = std::min(n_views - k0, kProjectViews);
    for (int k = 0; k < c; ++k)
      views.v[k] = {make_cam(&cams[k0 + k]), (float4*)splat[k0 + k], depth[k0 + k], radius[k0 + k],
                    (int4*)rect[k0 + k], clamp[k0 + k], g2d_clear != nullptr ? g2d_clear[k0 + k] : nullptr};
    launch_project<float>(params, n, c, views, rp, nullptr, as_stream(stream));
  }
  return hip_status(who);
}

extern "C" int32_t tgs_project(const float* params, int64_t n, const tgs_camera* cam,
                               const tgs_raster_params* rp, float* splat, float* depth,
                               int32_t* radius, int32_t* rect, uint8_t* clamp, float* g2d_clear,
                               void* stream) {
  TGS_REQUIRE(n >= 0, "tgs_project: n < 0");
  TGS_REQUIRE(cam != nullptr && cam->width > 0 && cam->height > 0, "tgs_project: bad camera");
  if (int32_t e = check_raster_params(rp)) return e;
  if (n == 0) return TGS_OK;
  TGS_REQUIRE(params && splat && depth && radius && rect && clamp, "tgs_project: null pointer");
  TGS_REQUIRE(((uintptr_t)splat & 15) == 0 && ((uintptr_t)rect & 15) == 0,
              "tgs_project: splat and rect must be 16-byte aligned");
  ProjectViews views{};
  views.v[0] = {make_cam(cam), (float4*)splat, depth, radius, (int4*)rect, clamp, g2d_clear};
  launch_project<float>(params, n, 1, views, rp, nullptr, as_stream(stream));
  return hip_status("tgs_project");
}

extern "C" int32_t tgs_project_bwd(const float* params, int64_t n, const tgs_camera* cam,
                                   const tgs_raster_params* rp, const int32_t* radius,
                                   const uint8_t* clamp, const float* g2d, float* grad,
                                   int32_t accumulate, void* stream) {
  TGS_REQUIRE(n >= 0, "tgs_project_bwd: n < 0");
  TGS_REQUIRE(cam != nullptr && cam->width > 0 && cam->height > 0, "tgs_project_bwd: bad camera");
  if (int32_t e = check_raster_params(rp)) return e;
  if (n == 0) return TGS_OK;
  TGS_REQUIRE(params && radius && clamp && g2d && grad, "tgs_project_bwd: null pointer");
  launch_project_bwd<float>(params, n, cam, rp, radius, clamp, g2d, grad, accumulate != 0, as_stream(stream));
  return hip_status("tgs_project_bwd");
}

// ---- FP64 instantiation (gradient checks): the same kernels over double
// parameters; the float outputs feed tgs_bin_sort as usual.
extern "C" int32_t tgs_project_f64(const double* params, int64_t n, const tgs_camera* cam,
                                   const tgs_raster_params* rp, double* rec64, float* splat, float* depth,
                                   int32_t* radius, int32_t* rect, uint8_t* clamp, void* stream) {
  TGS_REQUIRE(n >= 0, "tgs_project_f64: n < 0");
  TGS_REQUIRE(cam != nullptr && cam->width > 0 && cam->height > 0, "tgs_project_f64: bad camera");
  if (int32_t e = check_raster_params(rp)) return e;
  if (n == 0) return TGS_OK;
  TGS_REQUIRE(params && rec64 && splat && depth && radius && rect && clamp, "tgs_project_f64: null pointer");
  TGS_REQUIRE(((uintptr_t)splat & 15) == 0 && ((uintptr_t)rect & 15) == 0,
              "tgs_project_f64: splat and rect must be 16-byte aligned");
  ProjectViews views{};
  views.v[0] = {make_cam(cam), (float4*)splat, depth, radius, (int4*)rect, clamp, nullptr};
  launch_project<double>(params, n, 1, views, rp, rec64, as_stream(stream));
  return hip_status("tgs_project_f64");
}

extern "C" int32_t tgs_project_bwd_f64(const double* params, int64_t n, const tgs_camera* cam,
                                       const tgs_raster_params* rp, const int32_t* radius, const uint8_t* clamp,
                                       const double* g2d, double* grad, int32_t accumulate, void* stream) {
  TGS_REQUIRE(n >= 0, "tgs_project_bwd_f64: n < 0");
  TGS_REQUIRE(cam != nullptr && cam->width > 0 && cam->height > 0, "tgs_project_bwd_f64: bad camera");
  if (int32_t e = check_raster_params(rp)) return e;
  if (n == 0) return TGS_OK;
  TGS_REQUIRE(params && radius && clamp && g2d && grad, "tgs_project_bwd_f64: null pointer");
  launch_project_bwd<double>(params, n, cam, rp, radius, clamp, g2d, grad, accumulate != 0, as_stream(stream));
  return hip_status("tgs_project_bwd_f64");
}
