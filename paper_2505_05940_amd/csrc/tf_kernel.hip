// Transfer-function response of linear modal systems and its gradient
// (gfx950, float-float arithmetic on FP32 pairs split from FP64 inputs).
//
// With impulse invariance each mode is the discrete system
// b1 z / (z^2 + a1 z + a2) (paper: Sec. 3.2, transfer function); the linear
// string fits of Sec. 4.3 add a second numerator coefficient b2 per mode and
// free output weights w, and compare the magnitude response on a Bark-scale
// frequency grid with the target's spectral envelope:
//   H_b(e^{i Omega_k}) = sum_{mu of b} w_mu (b1_mu z + b2_mu) / (z^2 + a1_mu z + a2_mu).
// Coefficients per mode are (a1, a2, b1, b2, w).
//
// tf_response: 16 frequencies a workgroup, the modes of each spread over 16
// lanes.  tf_grad: a workgroup per mode, threads over the frequencies, for
// L = sum_k Re(conj(g_k) H_k): with N = b1 z + b2, D = z^2 + a1 z + a2,
//   dH/dw = N/D, dH/db1 = w z/D, dH/db2 = w/D, dH/da1 = -w N z/D^2,
//   dH/da2 = -w N/D^2.
// A call is bound by its latency (one allocation, a copy each way, a launch):
// 40 modes at 512 frequencies took 45 us with one thread a frequency and 22 us
// with one wave a mode.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.h"

namespace modal {

namespace {

// Error-free transformations (Knuth's TwoSum, Dekker's Fast2Sum, and the
// FMA-based exact product).  This file is compiled with -ffp-contract=off so
// only the explicit fmaf calls fuse.
struct ff {
  float hi, lo;
};
__device__ __forceinline__ ff two_sum(float a, float b) {
  float s = a + b;
  float bb = s - a;
  float e = (a - (s - bb)) + (b - bb);
  return {s, e};
}
__device__ __forceinline__ ff fast_two_sum(float a, float b) {
  float s = a + b;
  float e = b - (s - a);
  return {s, e};
}
__device__ __forceinline__ ff two_prod(float a, float b) {
  const float p = a * b;
  return {p, fmaf(a, b, -p)};
}
__device__ __forceinline__ ff ff_add(ff a, ff b) {
  ff s = two_sum(a.hi, b.hi);
  ff t = two_sum(a.lo, b.lo);
  float e = s.lo + t.hi;
  s = fast_two_sum(s.hi, e);
  e = s.lo + t.lo;
  return fast_two_sum(s.hi, e);
}
__device__ __forceinline__ ff ff_mul(ff a, ff b) {
  float p = a.hi * b.hi;
  float e = fmaf(a.hi, b.hi, -p);
  e = fmaf(a.hi, b.lo, e);
  e = fmaf(a.lo, b.hi, e);
  return fast_two_sum(p, e);
}
__device__ __forceinline__ ff ff_mul_f(ff a, float b) {
  float p = a.hi * b;
  float e = fmaf(a.hi, b, -p);
  e = fmaf(a.lo, b, e);
  return fast_two_sum(p, e);
}

__device__ __forceinline__ ff fneg(ff a) { return {-a.hi, -a.lo}; }
__device__ __forceinline__ ff fsub(ff a, ff b) { return ff_add(a, fneg(b)); }

// a / b to about float-float precision: two correction steps on the FP32
// quotient of the high parts
__device__ __forceinline__ ff fdiv(ff a, ff b) {
  const float q1 = a.hi / b.hi;
  ff r = fsub(a, ff_mul_f(b, q1));
  const float q2 = r.hi / b.hi;
  r = fsub(r, ff_mul_f(b, q2));
  const float q3 = r.hi / b.hi;
  const ff q = fast_two_sum(q1, q2);
  return ff_add(q, {q3, 0.f});
}

struct cx {
  ff re, im;
};
__device__ __forceinline__ cx cmul(cx x, cx y) {
  return {fsub(ff_mul(x.re, y.re), ff_mul(x.im, y.im)), ff_add(ff_mul(x.re, y.im), ff_mul(x.im, y.re))};
}
__device__ __forceinline__ cx cadd(cx x, cx y) { return {ff_add(x.re, y.re), ff_add(x.im, y.im)}; }
__device__ __forceinline__ cx cscale(cx x, ff s) { return {ff_mul(x.re, s), ff_mul(x.im, s)}; }
// 1 / d = conj(d) / |d|^2
__device__ __forceinline__ cx cinv(cx d) {
  const ff n = ff_add(ff_mul(d.re, d.re), ff_mul(d.im, d.im));
  return {fdiv(d.re, n), fdiv(fneg(d.im), n)};
}
__device__ __forceinline__ ff split(double v) {
  const float h = (float)v;
  return {h, (float)(v - (double)h)};
}
__device__ __forceinline__ double join(ff v) { return (double)v.hi + (double)v.lo; }
__device__ __forceinline__ cx point(double omega) {
  double s, c;
  sincos(omega, &s, &c);
  return {split(c), split(s)};
}
// Re(conj(g) v)
__device__ __forceinline__ ff re_dot(cx g, cx v) { return ff_add(ff_mul(g.re, v.re), ff_mul(g.im, v.im)); }
// sums over groups of W lanes
template <int W>
__device__ __forceinline__ ff lanes_sum(ff v) {
#pragma unroll
  for (int o = 1; o < W; o *= 2) v = ff_add(v, {__shfl_xor(v.hi, o, W), __shfl_xor(v.lo, o, W)});
  return v;
}

constexpr int kTfFreqs = 16, kTfLanes = 16;  // frequencies per workgroup, lanes over modes
constexpr int kTfThreads = 256;              // threads of a mode's gradient
constexpr int kTfBlocks = 1 << 23;           // workgroups along x of a launch: 2^31 threads, a grid takes under 2^32

}  // namespace

__global__ void __launch_bounds__(kTfFreqs* kTfLanes) tf_response_kernel(const double* __restrict__ coef,
                                                                         const int* __restrict__ mode_off,
                                                                         const double* __restrict__ omega, int k0,
                                                                         int n_freq, double2* __restrict__ H) {
  const int i = blockIdx.x * kTfFreqs + threadIdx.x / kTfLanes, left = n_freq - k0, ml = threadIdx.x % kTfLanes;
  const int k = k0 + min(i, left - 1);
  const int b = blockIdx.y;
  const cx z = point(omega[k]), z2 = cmul(z, z);
  const ff zero = {0.f, 0.f};
  cx acc = {zero, zero};
  for (int m = mode_off[b] + ml; m < mode_off[b + 1]; m += kTfLanes) {
    const double* c = coef + 5LL * m;
    const cx N = cadd(cscale(z, split(c[2])), cx{split(c[3]), zero});
    const cx D = cadd(z2, cadd(cscale(z, split(c[0])), cx{split(c[1]), zero}));
    acc = cadd(acc, cscale(cmul(N, cinv(D)), split(c[4])));
  }
  acc = {lanes_sum<kTfLanes>(acc.re), lanes_sum<kTfLanes>(acc.im)};
  if (ml == 0 && i < left) H[(long long)b * n_freq + k] = make_double2(join(acc.re), join(acc.im));
}

__global__ void __launch_bounds__(kTfThreads) tf_grad_kernel(const double* __restrict__ coef,
                                                             const int* __restrict__ mode_off,
                                                             const double* __restrict__ omega, int m0, int n_freq,
                                                             const double2* __restrict__ gH,
                                                             double* __restrict__ g_coef) {
  __shared__ float2 part[kTfThreads / kWave][5];
  const int b = blockIdx.y;
  const int i = m0 + blockIdx.x;
  if (i >= mode_off[b + 1] - mode_off[b]) return;
  const int m = mode_off[b] + i;
  const double* c = coef + 5LL * m;
  const ff zero = {0.f, 0.f};
  const ff a1 = split(c[0]), a2 = split(c[1]), b1 = split(c[2]), b2 = split(c[3]), w = split(c[4]);
  ff g[5] = {zero, zero, zero, zero, zero};
  for (int k = threadIdx.x; k < n_freq; k += kTfThreads) {
    const cx z = point(omega[k]), z2 = cmul(z, z);
    const cx N = cadd(cscale(z, b1), cx{b2, zero});
    const cx iD = cinv(cadd(z2, cadd(cscale(z, a1), cx{a2, zero})));
    const cx ND = cmul(N, iD), ND2 = cmul(ND, iD);
    const double2 G2 = gH[(long long)b * n_freq + k];
    const cx G = {split(G2.x), split(G2.y)};
    g[0] = ff_add(g[0], fneg(ff_mul(re_dot(G, cmul(ND2, z)), w)));
    g[1] = ff_add(g[1], fneg(ff_mul(re_dot(G, ND2), w)));
    g[2] = ff_add(g[2], ff_mul(re_dot(G, cmul(iD, z)), w));
    g[3] = ff_add(g[3], ff_mul(re_dot(G, iD), w));
    g[4] = ff_add(g[4], re_dot(G, ND));
  }
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    const ff v = lanes_sum<kWave>(g[i]);
    if (threadIdx.x % kWave == 0) part[threadIdx.x / kWave][i] = make_float2(v.hi, v.lo);
  }
  __syncthreads();
  if (threadIdx.x < 5) {
    ff s = zero;
    for (int v = 0; v < kTfThreads / kWave; ++v) s = ff_add(s, {part[v][threadIdx.x].x, part[v][threadIdx.x].y});
    g_coef[5LL * m + threadIdx.x] = join(s);
  }
}

hipError_t launch_tf_response(const double* coef, const int* mode_off, int batch, const double* omega, int n_freq,
                              double2* H, hipStream_t s) {
  for (int k0 = 0, n; k0 < n_freq; k0 += n) {
    n = std::min(n_freq - k0, kTfBlocks * kTfFreqs);
    hipLaunchKernelGGL(tf_response_kernel, dim3((n + kTfFreqs - 1) / kTfFreqs, batch), dim3(kTfFreqs * kTfLanes), 0, s,
                       coef, mode_off, omega, k0, n_freq, H);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_tf_grad(const double* coef, const int* mode_off, int batch, int max_modes, const double* omega,
                          int n_freq, const double2* gH, double* g_coef, hipStream_t s) {
  for (int m0 = 0, n; m0 < max_modes; m0 += n) {
    n = std::min(max_modes - m0, kTfBlocks);
    hipLaunchKernelGGL(tf_grad_kernel, dim3(n, batch), dim3(kTfThreads), 0, s, coef, mode_off, omega, m0, n_freq, gH,
                       g_coef);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace modal
