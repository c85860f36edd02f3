// Light baking (Sec. 3.4, "Light Baking", Eq. 10): the per-surfel radiance r
// is refitted so that the 0-bounce image (R composited along the camera ray,
// Sec. 3.2) matches path-traced renders, min_r L1(PQ(L0), PQ(Lpt)).
//
// k_zero_bounce        one work item per pixel on the persistent segment
//                      runner: the camera ray through the pixel (sample 0),
//                      blending r only; writes R.
// k_zero_bounce_adj_r  the same rays re-traced: every blended hit adds
//                      w_i dL to its surfel's radiance gradient (L0 is linear
//                      in r, with weights w_i = T_{i-1} alpha_i that do not
//                      depend on it); double atomics into the workspace, the
//                      three of a hit by neighbouring lanes (add_rows).
// k_bake_loss          per value: |PQ(L0) - PQ(Lpt)| (summed per block, then
//                      one double atomic per block) and its derivative
//                      sign * PQ'(L0) / count.
// k_adam               Adam with bias correction on r, then r clamped at 0.
//
// PQ is SMPTE ST 2084 on Y = max(L, 0) / 10000 (radiance read as cd/m^2),
// its derivative taken at max(Y, 2^-24); double precision throughout.
#include "eag_device.h"
#include "eag_internal.h"
#include "eag_render.h"
#include "eag_runner.h"

#include <algorithm>
#include <cmath>

namespace eag {

namespace {

constexpr double PQ_M1 = 2610.0 / 16384.0;
constexpr double PQ_M2 = 2523.0 / 4096.0 * 128.0;
constexpr double PQ_C1 = 3424.0 / 4096.0;
constexpr double PQ_C2 = 2413.0 / 4096.0 * 32.0;
constexpr double PQ_C3 = 2392.0 / 4096.0 * 32.0;
constexpr double PQ_PEAK = 10000.0;
constexpr double PQ_YMIN = 5.9604644775390625e-08;   // 2^-24

__device__ __forceinline__ double pq_curve(double L) {
  const double ym = pow(fmax(L, 0.0) / PQ_PEAK, PQ_M1);
  return pow((PQ_C1 + PQ_C2 * ym) / (1.0 + PQ_C3 * ym), PQ_M2);
}

__device__ __forceinline__ double pq_slope(double L) {
  if (L < 0.0) return 0.0;
  const double y = fmax(L / PQ_PEAK, PQ_YMIN);
  const double ym = pow(y, PQ_M1);
  const double num = PQ_C1 + PQ_C2 * ym, den = 1.0 + PQ_C3 * ym;
  const double dbase = (PQ_C2 * den - PQ_C3 * num) / (den * den);
  return PQ_M2 * pow(num / den, PQ_M2 - 1.0) * dbase * (PQ_M1 * ym / y) / PQ_PEAK;
}

struct ZeroBounceSource {
  const CamBatch* cams;
  int64_t hw;
  SbParams sp;
  float* rgb;
  int64_t item;

  static constexpr bool kHits = false;
  __device__ __forceinline__ void operator()(const Record&, const Attr&, double, double, double, double, D3, D3) const {}

  __device__ __forceinline__ bool start(int64_t wid, TraceCtx&, D3& O, D3& W) {
    item = wid;
    const CamDev& c = cams->c[wid / hw];
    O = d3(c.eye[0], c.eye[1], c.eye[2]);
    W = pixel_dir(c, (uint32_t)(wid % hw), 0, sp.flags, sp.k0, sp.k1);
    return true;
  }

  __device__ __forceinline__ bool finish(const Seg<false>& s, D3&, D3&) {
    rgb[item * 3 + 0] = s.R0;
    rgb[item * 3 + 1] = s.R1;
    rgb[item * 3 + 2] = s.R2;
    return false;
  }
};

template <bool GROUPS>
__global__ void __launch_bounds__(TRACE_BLOCK) __attribute__((amdgpu_waves_per_eu(2))) k_zero_bounce(TraceCtx tc, const CamBatch cams, int64_t hw,
                                                            int32_t n_cams, SbParams sp, float* rgb,
                                                            unsigned long long* work, uint64_t* hitlist) {
  ZeroBounceSource src;
  src.cams = &cams;
  src.hw = hw;
  src.sp = sp;
  src.rgb = rgb;
  src.item = 0;
  run_work<GROUPS, Q_RADIANCE, false, false>(tc, src, work, hw * n_cams, hitlist, nullptr);
}

using RadAdds = RowAdds<3, 64>;
struct RadianceAdjSource {
  const CamBatch* cams;
  int64_t hw;
  SbParams sp;
  const float* dL;
  double* gr;          // [n][RAD_STRIDE] accumulators
  RadAdds* adds;       // this wave's, in LDS
  V3 dl;

  __device__ __forceinline__ bool start(int64_t wid, TraceCtx&, D3& O, D3& W) {
    dl = v3(dL[wid * 3 + 0], dL[wid * 3 + 1], dL[wid * 3 + 2]);
    if (dl.x == 0.0f && dl.y == 0.0f && dl.z == 0.0f) return false;   // nothing to add
    const CamDev& c = cams->c[wid / hw];
    O = d3(c.eye[0], c.eye[1], c.eye[2]);
    W = pixel_dir(c, (uint32_t)(wid % hw), 0, sp.flags, sp.k0, sp.k1);
    return true;
  }

  static constexpr bool kHits = true;
  double prefix = 0.0;   // (of nothing)
  __device__ __forceinline__ void operator()(const Record& r, const Attr& at, double t, double om, double w, double Tb, D3 O,
                                             D3 W) {
    adjoint(r, at, t, om, w, Tb, 0.0, 0.0, O, W);
  }
  __device__ __forceinline__ double weight(const Record&, const Attr&, double, D3) const { return 0.0; }
  __device__ __forceinline__ void gather(int, bool) {}
  __device__ __forceinline__ void leave() {}
  __device__ __forceinline__ void adjoint(const Record& r, const Attr&, double, double, double w, double, double, double, D3, D3) {
    const uint32_t idx = rec_index(r);
    const double v[3] = {w * (double)dl.x, w * (double)dl.y, w * (double)dl.z};
    add_rows(adds, gr, RAD_STRIDE, idx, v);
  }

  __device__ __forceinline__ bool finish(const Seg<false>&, D3&, D3&) { return false; }
};

template <bool GROUPS>
__global__ void __launch_bounds__(TRACE_BLOCK) __attribute__((amdgpu_waves_per_eu(2))) k_zero_bounce_adj_r(TraceCtx tc, const CamBatch cams, int64_t hw,
                                                                  int32_t n_cams, SbParams sp, const float* dL,
                                                                  double* gr, unsigned long long* work,
                                                                  uint64_t* hitlist) {
  RadianceAdjSource src;
  src.cams = &cams;
  src.hw = hw;
  src.sp = sp;
  src.dL = dL;
  __shared__ RadAdds s_adds[TRACE_BLOCK / 64];
  src.gr = gr;
  src.adds = s_adds + (threadIdx.x >> 6);
  src.dl = v3(0.f, 0.f, 0.f);
  run_work<GROUPS, Q_RADIANCE, false, false>(tc, src, work, hw * n_cams, hitlist, nullptr);
}

// Grid-stride: one loss atomic per block, all on one address (with a block per
// 256 of the 4.7 M values of 8 views at 512x384 they set the time, 0.27 ms).
__global__ void __launch_bounds__(256) k_bake_loss(const float* rgb, const float* target, int64_t m, double inv_count,
                                                  float* dL, double* loss) {
  __shared__ double part[256 / 64];
  double a = 0.0;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < m; i += (int64_t)gridDim.x * blockDim.x) {
    const double l0 = rgb[i];
    const double d = pq_curve(l0) - pq_curve((double)target[i]);
    a += fabs(d);
    const double sg = d > 0.0 ? 1.0 : (d < 0.0 ? -1.0 : 0.0);
    dL[i] = (float)(sg * pq_slope(l0) * inv_count);
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) a += __shfl_xor(a, o);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = a;
  __syncthreads();
  if (threadIdx.x == 0) atomicAdd(loss, (part[0] + part[1] + part[2] + part[3]) * inv_count);
}

__device__ __forceinline__ void adam_update(float* r, float gi, float* m, float* v, int64_t i, float lr, float b1,
                                            float b2, float eps, float c1, float c2) {
  const float mi = b1 * m[i] + (1.0f - b1) * gi;
  const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  // c1 = 1 - b1^step, c2 = 1 - b2^step
  const float step = lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  r[i] = fmaxf(r[i] - step, 0.0f);
}

__global__ void k_adam(float* r, const float* g, float* m, float* v, int64_t count, float lr, float b1, float b2,
                       float eps, float c1, float c2) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < count) adam_update(r, g[i], m, v, i, lr, b1, b2, eps, c1, c2);
}

// The three components of surfel j from its accumulator row.
__device__ __forceinline__ void load_rad(const double* acc, int64_t j, float (&g)[3]) {
  const double2 a = reinterpret_cast<const double2*>(acc)[2 * j], b = reinterpret_cast<const double2*>(acc)[2 * j + 1];
  g[0] = (float)a.x;
  g[1] = (float)a.y;
  g[2] = (float)b.x;
}

__global__ void k_adam_radiance(float* r, const double* acc, float* m, float* v, int64_t n, float lr, float b1,
                                float b2, float eps, float c1, float c2) {
  const int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (j >= n) return;
  float g[3];
  load_rad(acc, j, g);
#pragma unroll
  for (int k = 0; k < 3; ++k) adam_update(r, g[k], m, v, k * n + j, lr, b1, b2, eps, c1, c2);
}

__global__ void k_add_grad(const double* acc, int64_t n, float* g) {
  const int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (j >= n) return;
  float v[3];
  load_rad(acc, j, v);
#pragma unroll
  for (int k = 0; k < 3; ++k) g[k * n + j] += v[k];
}

__global__ void k_zero_f64_b(double* p, int64_t count) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < count) p[i] = 0.0;
}

unsigned blocks_for(int64_t count) { return (unsigned)((count + 255) / 256); }

}  // namespace

void launch_zero_bounce(const TraceCtx& tc, const CamBatch& cams, int64_t hw, int32_t n_cams, const SbParams& sp,
                        float* rgb, unsigned long long* work, uint64_t* hitlist, hipStream_t st) {
  launch_zero_u64(work, 1, st);
  hipLaunchKernelGGL(by_groups(CAMERA, hw * n_cams, runner_lanes(), tc.idx_bits) ? k_zero_bounce<true> : k_zero_bounce<false>,
                     dim3((unsigned)(runner_lanes() / TRACE_BLOCK)), dim3(TRACE_BLOCK), 0, st, tc, cams, hw, n_cams, sp, rgb, work, hitlist);
  check_hip(hipGetLastError(), "zero-bounce launch");
}

void launch_zero_bounce_adj_r(const TraceCtx& tc, const CamBatch& cams, int64_t hw, int32_t n_cams,
                              const SbParams& sp, const float* dL, double* gacc, unsigned long long* work,
                              uint64_t* hitlist, hipStream_t st) {
  launch_zero_u64(work, 1, st);
  hipLaunchKernelGGL(by_groups(ADJOINTS, hw * n_cams, runner_lanes(), tc.idx_bits) ? k_zero_bounce_adj_r<true> : k_zero_bounce_adj_r<false>,
                     dim3((unsigned)(runner_lanes() / TRACE_BLOCK)), dim3(TRACE_BLOCK), 0, st, tc, cams, hw, n_cams, sp, dL, gacc, work, hitlist);
  check_hip(hipGetLastError(), "zero-bounce adjoint launch");
}

void launch_zero_f64(double* p, int64_t count, hipStream_t st) {
  if (count > 0) hipLaunchKernelGGL(k_zero_f64_b, dim3(blocks_for(count)), dim3(256), 0, st, p, count);
}

void launch_add_grad(const double* acc, int64_t n, float* g, hipStream_t st) {
  if (n > 0) hipLaunchKernelGGL(k_add_grad, dim3(blocks_for(n)), dim3(256), 0, st, acc, n, g);
}

void launch_bake_loss(const float* rgb, const float* target, int64_t m, float* dL, double* loss, hipStream_t st) {
  launch_zero_f64(loss, 1, st);
  if (m > 0)
    hipLaunchKernelGGL(k_bake_loss, dim3(std::min(blocks_for(m), 1024u)), dim3(256), 0, st, rgb, target, m, 1.0 / (double)m, dL, loss);
  check_hip(hipGetLastError(), "bake loss launch");
}

namespace {
void adam_corrections(const eag_adam& a, int32_t step, float& c1, float& c2) {
  c1 = (float)(1.0 - std::pow((double)a.beta1, step));
  c2 = (float)(1.0 - std::pow((double)a.beta2, step));
}
}  // namespace

void launch_adam_radiance(float* r, const double* acc, float* m, float* v, int64_t n, const eag_adam& a, int32_t step,
                          hipStream_t st) {
  float c1, c2;
  adam_corrections(a, step, c1, c2);
  if (n > 0)
    hipLaunchKernelGGL(k_adam_radiance, dim3(blocks_for(n)), dim3(256), 0, st, r, acc, m, v, n, a.lr, a.beta1, a.beta2,
                       a.eps, c1, c2);
  check_hip(hipGetLastError(), "adam launch");
}

void launch_adam(float* r, const float* g, float* m, float* v, int64_t count, const eag_adam& a, int32_t step,
                 hipStream_t st) {
  float c1, c2;
  adam_corrections(a, step, c1, c2);
  if (count > 0)
    hipLaunchKernelGGL(k_adam, dim3(blocks_for(count)), dim3(256), 0, st, r, g, m, v, count, a.lr, a.beta1, a.beta2,
                       a.eps, c1, c2);
  check_hip(hipGetLastError(), "adam launch");
}

}  // namespace eag
