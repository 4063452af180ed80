// Time-parallel evaluation of linear modal systems (gfx950, FP64 matrix cores).
//
// Without a nonlinear force each mode of the recursion of the modal
// oscillator update (paper: Sec. 3.2), q^{n+1} = g q^n + p q^{n-1} + r f^n,
// is solved in closed form by the roots z1, z2 of z^2 - g z - p: the free
// response is A z1^n + B z2^n, and a unit force at step m adds
// h(n - m) = C (z1^(n-m) - z2^(n-m)), C = r / (z1 - z2), for n > m.  The paper
// evaluates such responses by repeated multiplication with the discrete
// eigenvalues in a prefix sum over time (Sec. 4.3, linear string fits).
//
// Here every output sample of every mode is a value Re(P1 z1^n + P2 z2^n)
// for one of three amplitude sets:
//   free   (P1, P2) = c (A, B),         exponent n, every step before the
//                                        excitation ends (and all steps of an
//                                        unforced instance);
//   post   (P1, P2) = c (V1, V2),       exponent n - n_exc, every step from
//                                        n_exc on, where Vk = A z_k^{n_exc} +
//                                        b C sum_{m < n_exc} e[m] z_k^{n_exc - m}
//                                        (the state the excitation leaves);
//   impulse(P1, P2) = c b C (1, -1),    exponent = lag, the output-space impulse
//                                        response used inside the excitation
//                                        window.
// A complex-conjugate pair keeps one root z with the amplitude P doubled; a
// real pair keeps both.
//
// lin_sum: sample n0 + 64 a + b is a contraction over the modes,
//   y[a][b] = sum_modes Re(P z^n0 (z^64)^a) Re(z^b) - Im(P z^n0 (z^64)^a) Im(z^b)
// (for a real pair the two roots take the places of the two parts), which is
// a matrix product: two columns of A and two rows of B per mode, on
// v_mfma_f64_16x16x4f64.  Lane l supplies A[l % 16][l / 16] and
// B[l / 16][l % 16] and receives D[4 r + l / 16][l % 16] in accumulator r
// (checked on the device).  A wave owns 16 FR rows of 64 samples; z^b and
// (z^64)^a come from tables built once, z^n0 by binary exponentiation for 64
// modes at a time, one per lane.  Column tile j of lane column c is sample
// 4 c + j, so that a lane ends with four consecutive samples of a row.
//
// 2 048 strings, 70 690 modes, 44 100 samples (1.25e10 products): the
// float-float recurrence on the vector ALU took 3.4 ms, this 0.36.  The
// products alone take 0.165 ms at the FP64 matrix rate (78.6 TFLOP/s) and the
// 361 MB of outputs 0.08; the tables (4 KB of cache reads a wave and 512
// matrix cycles) are read two mode pairs ahead.  With the factors of a pair
// broadcast by lane reads and selected, 93 vector instructions for 8 matrix
// ones, it took 0.40 ms; rows of 64 a wave (one wave per SIMD) 0.50.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device_common.h"
#include "kernels.h"

namespace modal {

typedef double v4d __attribute__((ext_vector_type(4)));

namespace {

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x));
}

// z^n, n >= 0, by binary exponentiation
__device__ __forceinline__ double2 cpow(double2 z, long long n) {
  double2 r = make_double2(1., 0.);
  while (n > 0) {
    if (n & 1) r = cmul(r, z);
    n >>= 1;
    if (n > 0) z = cmul(z, z);
  }
  return r;
}

__device__ __forceinline__ double rpow(double z, long long n) {
  double r = 1.;
  while (n > 0) {
    if (n & 1) r *= z;
    n >>= 1;
    z *= z;
  }
  return r;
}

// (z^n of a conjugate pair's root) or (z1^n, z2^n) of a real pair
__device__ __forceinline__ double2 mode_pow(const LinMode& m, long long n) {
  if (m.conj) return cpow(m.z1, n);
  return make_double2(rpow(m.z1.x, n), rpow(m.z2.x, n));
}

// The run of samples of one workgroup row: [i0, i0 + len) of out from
// exponent e0 of an amplitude set.
struct Run {
  int set;
  long long e0, len, out;
};

}  // namespace

// blockIdx.y < batch: instance blockIdx.y's free response over [base, base + n)
// up to the end of its excitation (to the end if it has none); from batch on:
// forced instance blockIdx.y - batch's response to the state that the
// excitation left.  With impulse set, the impulse response of forced instance
// blockIdx.y at lags 1, 2, ...
template <int FR, typename OutT>
__global__ void __launch_bounds__(kWave* kLinWaves) lin_sum_kernel(LinParams P, OutT* __restrict__ out) {
  const int y = blockIdx.y;
  const bool post = !P.impulse && y >= P.batch;
  const int b = P.impulse ? (int)P.forced[y].inst : (post ? (int)P.forced[y - P.batch].inst : y);
  const LinInst I = P.inst[b];
  Run r;
  if (P.impulse) {
    r = {2, 1, I.n_exc - 1, y * P.out_stride};
  } else if (!post) {
    const long long end = I.n_exc > 0 ? min(P.base + P.n, I.n_exc) : P.base + P.n;
    r = {0, P.base, end - P.base, b * P.out_stride};
  } else {
    const long long p0 = max(P.base, I.n_exc);
    r = {1, p0 - I.n_exc, P.base + P.n - p0, b * P.out_stride + (p0 - P.base)};
  }
  // per wave, the factors of (z^64)^a's two parts in both columns of A of a
  // group's modes: [mode][column]
  __shared__ double2 fac[kLinWaves][128];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform
  const long long s0 = ((long long)blockIdx.x * kLinWaves + wave) * (kLinCols * 16 * FR);
  if (s0 >= r.len) return;
  const int row = lane & 15, q = lane >> 4;  // A row and K index; B column group and K index
  const int so = (q >> 1) * 32 + row;                // this lane's entry of a pair's tables
  const int zo = q * kLinCols + 4 * row;
  const double2* amp = P.amp + (long long)r.set * P.modes;
  v4d acc[FR][4];
#pragma unroll
  for (int f = 0; f < FR; ++f)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[f][j] = (v4d){0., 0., 0., 0.};
  for (int kb = I.m0; kb < I.m1; kb += 64) {
    const int kl = min(kb + lane, I.m1 - 1);
    const LinMode md = P.mode[kl];
    const double2 w = mode_pow(md, r.e0 + s0), p = amp[kl];  // P z^(e0 + s0) of mode kb + lane
    const double2 u = md.conj ? cmul(p, w) : make_double2(p.x * w.x, p.y * w.y);
    const bool in = kb + lane < I.m1;
    wave_lds_sync();  // the previous group's factors are read
    fac[wave][2 * lane] = make_double2(in ? u.x : 0., in && md.conj ? -u.y : 0.);
    fac[wave][2 * lane + 1] = make_double2(in && md.conj ? -u.y : 0., in ? (md.conj ? -u.x : u.y) : 0.);
    wave_lds_sync();
    const int pairs = (min(64, I.m1 - kb) + 1) / 2;
    const double2* s64 = P.s64 + (long long)kb * 32;
    const double* zt = P.z + (long long)kb * 2 * kLinCols;
    // tables of this lane's mode of pair i, read two pairs ahead (they end in
    // eight modes of zeros, and past an instance's last mode the factors are
    // zero)
    struct Tab {
      double2 s[FR];
      v2d z[2];
      double2 c;  // factors of mode 2 i + q / 2, column q % 2
    };
    auto load = [&](Tab& t, int i) {
#pragma unroll
      for (int f = 0; f < FR; ++f) t.s[f] = (s64 + 64 * i)[so + 16 * f];
      const v2d* z = reinterpret_cast<const v2d*>(zt + 4 * kLinCols * i + zo);
      t.z[0] = z[0];
      t.z[1] = z[1];
      t.c = fac[wave][(4 * i + q) & 127];
    };
    auto mul = [&](Tab& t, int i) {
      const double2 c = t.c;
      double z[4] = {t.z[0].x, t.z[0].y, t.z[1].x, t.z[1].y};
      double av[FR];
#pragma unroll
      for (int f = 0; f < FR; ++f) av[f] = fma(c.x, t.s[f].x, c.y * t.s[f].y);
      __builtin_amdgcn_sched_barrier(0);
      load(t, i + 2);
      __builtin_amdgcn_sched_barrier(0);  // issued here, before the products
#pragma unroll
      for (int f = 0; f < FR; ++f)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[f][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[f], z[j], acc[f][j], 0, 0, 0);
    };
    Tab ta, tb;
    load(ta, 0);
    load(tb, 1);
    for (int i = 0; i < pairs; i += 2) {
      mul(ta, i);
      mul(tb, i + 1);  // (past the last pair, zeros)
    }
  }
  OutT* o = out + r.out + s0;
  const long long left = r.len - s0;
  const bool aligned = (reinterpret_cast<unsigned long long>(o) & (4 * sizeof(OutT) - 1)) == 0;
#pragma unroll
  for (int f = 0; f < FR; ++f)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const long long i = kLinCols * (16 * f + 4 * t + q) + 4 * row;
      if constexpr (sizeof(OutT) == 4) {
        if (aligned && i + 3 < left) {
          st4(reinterpret_cast<float*>(o) + i, make_float4((float)acc[f][0][t], (float)acc[f][1][t], (float)acc[f][2][t], (float)acc[f][3][t]));
          continue;
        }
      }
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (i + j < left) o[i + j] = (OutT)acc[f][j][t];
    }
}

// Tables of every mode: z[k][2][64], the real and imaginary parts of z^b (the
// powers of the two roots of a real pair), and s64[k][32] = (z^64)^a.
__global__ void lin_tab_kernel(const LinMode* __restrict__ modes, int M, double* __restrict__ z,
                               double2* __restrict__ s64) {
  const long long n = (long long)M * (kLinCols + 32), step = (long long)gridDim.x * blockDim.x;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += step) {
    const long long k = i / (kLinCols + 32);
    const int t = (int)(i % (kLinCols + 32));
    if (t < kLinCols) {
      const double2 v = mode_pow(modes[k], t);
      z[(2 * k) * kLinCols + t] = v.x;
      z[(2 * k + 1) * kLinCols + t] = v.y;
    } else {
      s64[k * 32 + t - kLinCols] = mode_pow(modes[k], (long long)kLinCols * (t - kLinCols));
    }
  }
}

// Amplitude sets [free | post | impulse] of every mode; the post set runs the
// excitation through each root (V <- (V + b C e[m]) z), one thread per mode.
__global__ void lin_amp_kernel(const LinInit* __restrict__ init, const LinMode* __restrict__ modes, int M,
                               const float* __restrict__ e_ext, double2* __restrict__ amp) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= M) return;
  const LinInit I = init[k];
  const LinMode md = modes[k];
  const double2 bc = make_double2(I.C.x * I.b, I.C.y * I.b);
  const float* e = e_ext + I.e_off;
  double2 v1 = I.A, v2 = I.B;
  for (long long m = 0; m < I.n_exc; ++m) {
    const double em = e[m];
    v1 = cmul(make_double2(fma(bc.x, em, v1.x), fma(bc.y, em, v1.y)), md.z1);
    if (!md.conj) v2 = cmul(make_double2(fma(-bc.x, em, v2.x), fma(-bc.y, em, v2.y)), md.z2);
  }
  const double f = md.conj ? 2. * I.c : I.c;
  auto pair = [&](double2 p1, double2 p2) {
    return md.conj ? make_double2(f * p1.x, f * p1.y) : make_double2(f * p1.x, f * p2.x);
  };
  amp[k] = pair(I.A, I.B);
  amp[(size_t)M + k] = pair(v1, v2);
  amp[2 * (size_t)M + k] = pair(bc, make_double2(-bc.x, -bc.y));
}

// Inside the excitation window: y[n - base] += sum_{m < n} e[m] h[n - m] for
// n in [base, min(base + n_steps, n_exc)); the h row holds lags 1 .. n_exc - 1.
// A wave takes kLinConv = 256 consecutive n, four a lane, and stages 256
// samples of e, with the 512 lags they meet, in LDS at a time.  Four n against
// four m meet seven lags, of which the next four m share three: 16 products
// for four 16-byte reads (256 windows of 1000 steps: 37 us; with one n a
// lane and a read of h for each product 47).
__global__ void __launch_bounds__(kWave) lin_conv_kernel(const LinForced* __restrict__ forced,
                                                         const double* __restrict__ h, long long h_stride,
                                                         const float* __restrict__ e_ext, long long base,
                                                         long long n_steps, float* __restrict__ y,
                                                         long long y_stride) {
  __shared__ __align__(16) double hs[2 * kLinConv], es[kLinConv];
  const LinForced F = forced[blockIdx.y];
  const int t = threadIdx.x;
  const long long i0 = (long long)blockIdx.x * kLinConv, nb = base + i0;  // the wave's first n
  const long long end = min(base + n_steps, F.n_exc);
  if (nb >= end) return;
  const float* e = e_ext + F.e_off;
  const double* hb = h + blockIdx.y * h_stride - 1;  // hb[lag], lag >= 1
  double v[4] = {0., 0., 0., 0.};
  for (long long m0 = 0; m0 < min(nb + kLinConv, end) - 1; m0 += kLinConv) {
    // (n, m) meet at lag n - m; hs[l] holds lag nb - m0 - kLinConv + 1 + l
    const long long l0 = nb - m0 - kLinConv + 1;
    __syncthreads();
    for (int l = t; l < kLinConv; l += kWave) es[l] = m0 + l < F.n_exc ? (double)e[m0 + l] : 0.;
    for (int l = t; l < 2 * kLinConv; l += kWave) {
      const long long lag = l0 + l;
      hs[l] = lag >= 1 && lag < F.n_exc ? hb[lag] : 0.;
    }
    __syncthreads();
    // n = nb + 4 t + j and m = m0 + 4 u + k: lag index 4 (t - u) + 252 + (j - k + 3)
    f64x4 lo = ld4d(hs + 4 * t + kLinConv), hi;
#pragma unroll 4
    for (int u = 0; u < kLinConv / 4; ++u) {
      hi = lo;
      lo = ld4d(hs + 4 * (t - u) + kLinConv - 4);
      const f64x4 ev = ld4d(es + 4 * u);
      const double w[7] = {lo.v[0], lo.v[1], lo.v[2], lo.v[3], hi.v[0], hi.v[1], hi.v[2]};
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int k = 0; k < 4; ++k) v[j] = fma(ev.v[k], w[j - k + 3], v[j]);
    }
  }
  float* yo = y + F.inst * y_stride + i0 + 4 * t;
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if (nb + 4 * t + j < end) yo[j] = (float)((double)yo[j] + v[j]);
}

// Waves of 32 rows of 64 samples where the batch has enough of them to fill
// the chip, of 16 otherwise.
template <typename OutT>
static hipError_t lin_sum(const LinParams& P, int rows, long long max_len, OutT* out, hipStream_t s) {
  if (max_len < 1 || rows < 1) return hipSuccess;
  const long long waves = (max_len + 2 * 16 * kLinCols - 1) / (2 * 16 * kLinCols) * rows;
  const int fr = waves >= 2048 ? 2 : 1;
  const long long per_block = 16LL * fr * kLinCols * kLinWaves;
  dim3 grid((unsigned)((max_len + per_block - 1) / per_block), rows);
  if (fr == 2)
    hipLaunchKernelGGL((lin_sum_kernel<2, OutT>), grid, dim3(kWave * kLinWaves), 0, s, P, out);
  else
    hipLaunchKernelGGL((lin_sum_kernel<1, OutT>), grid, dim3(kWave * kLinWaves), 0, s, P, out);
  return hipGetLastError();
}

hipError_t launch_lin_sum(const LinParams& P, int n_forced, float* out, hipStream_t s) {
  return lin_sum<float>(P, P.batch + n_forced, P.n, out, s);
}

hipError_t launch_lin_impulse(const LinParams& P, int n_forced, long long max_len, double* out, hipStream_t s) {
  return lin_sum<double>(P, n_forced, max_len, out, s);
}

hipError_t launch_lin_init(const LinInit* init, const LinMode* modes, int M, const float* e_ext, double2* amp,
                           double* z, double2* s64, hipStream_t s) {
  if (M < 1) return hipSuccess;
  const long long tab_blocks = std::min(((kLinCols + 32LL) * M + 255) / 256, 1LL << 16);
  hipLaunchKernelGGL(lin_tab_kernel, dim3((unsigned)tab_blocks), dim3(256), 0, s, modes, M, z, s64);
  hipLaunchKernelGGL(lin_amp_kernel, dim3((M + 63) / 64), dim3(64), 0, s, init, modes, M, e_ext, amp);
  return hipGetLastError();
}

hipError_t launch_lin_conv(const LinForced* forced, int n_forced, const double* h, long long h_stride,
                           const float* e_ext, long long base, long long n_steps, long long window,
                           float* y, long long y_stride, hipStream_t s) {
  if (n_forced < 1 || window < 1) return hipSuccess;
  dim3 grid((unsigned)((window + kLinConv - 1) / kLinConv), n_forced);
  hipLaunchKernelGGL(lin_conv_kernel, grid, dim3(kWave), 0, s, forced, h, h_stride, e_ext, base, n_steps, y,
                     y_stride);
  return hipGetLastError();
}

}  // namespace modal
