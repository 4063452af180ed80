// Time loop for batches that share one parity-structured coupling tensor up to
// a per-row scale, the tensor in registers (gfx950, FP32 MFMA).
//
// As in shared_kernel.hip a step is, per in-plane row n, the product
// V0 = H0[n] X with the instances as columns, eta0 = column sums of V0 o X and
// F += s_n^2 eta0 V0.  A sine-family tensor's row n couples the modes of a
// class only to one partner class (class xor the row's pattern), so of the
// dense product three quarters are zeros.  Here the modes are grouped by
// class, one 16-row tile per class, and a tile multiplies its partner class
// only: 4 KS instructions v_mfma_f32_16x16x4f32 a row (KS = a class's 4-wide
// K steps), where the dense kernel issues kt kc: 12 against 30 at 40 modes.
// A workgroup of kScWaves waves owns 16 columns.  Each wave keeps R rows of
// one pattern with their A operands in registers for the whole launch, so no
// step stages or reads a tensor, and its B operands (the partner classes' X,
// in tile order) are the same for all its rows.  Per step
//   1. every wave reads X of its tiles from LDS as B operands and in
//      accumulator order, forms V0, eta0 and its partial F;
//   2. the partial forces meet in LDS (barrier), and every thread adds the
//      waves' partials of its two (mode, column) pairs, whose FP64 state and
//      coefficients it keeps in registers, advances them and publishes X
//      (barrier).  Outputs are summed over a wave's modes, collected in LDS
//      and written kScChunk steps at a time.
//
// Bound by the matrix cores' FP32 rate, two waves per SIMD, and by a step's
// serial part (LDS round trips and two barriers): at 40/40 a workgroup's step
// takes 4.0 us, of which the matrix instructions are 1.9.
#include <hip/hip_runtime.h>

#include "device_common.h"
#include "kernels.h"

namespace modal {

typedef float v4f __attribute__((ext_vector_type(4)));

template <int KS, int R>
__global__ void __launch_bounds__(kWave* kScWaves) shared_class_kernel(ScParams P) {
  constexpr int T = 4;                        // tiles, one per class
  constexpr int SLOTS = 16 * T;               // mode slots of a column
  constexpr int NP = SLOTS * 16 / (kWave * kScWaves);  // (slot, column) pairs per thread
  __shared__ __align__(16) float xs[SLOTS / 4][16][4];           // X[slot / 4][column][slot % 4]
  __shared__ __align__(16) float red[kScWaves][T][kWave][4];     // partial forces, accumulator order
  __shared__ float ys[kScChunk][kScWaves][16];                   // outputs, per wave's modes
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int col = lane & 15, quad = lane >> 4;
  const ScWg W = P.wg[blockIdx.x];
  const ScWave G = P.wave[W.group * kScWaves + wave];
  const SharedSlot sl = P.slot[blockIdx.x * 16 + col];

  // A[r][t][s]: lane l holds H0[row r][mode l % 16 of class t][mode 4 s + l / 16 of its partner]
  float A[R][T][KS], s2[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int s = 0; s < KS; ++s)
        A[r][t][s] = P.A[((((long long)W.group * kScWaves + wave) * R + r) * T * KS + t * KS + s) * kWave + lane];
    s2[r] = P.s2[(((long long)blockIdx.x * kScWaves + wave) * R + r) * 16 + col];
  }
  // this thread's pairs: column col, slots tid / 16 + 32 i
  double x[NP], d[NP], m[NP], p[NP], rr[NP];
  float bx[NP], cw[NP];
  const long long base_o = ((long long)blockIdx.x * 16 + col) * SLOTS + tid / 16;
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    const long long o = base_o + (kWave * kScWaves / 16) * i;
    x[i] = P.x[o];
    d[i] = P.d[o];
    m[i] = P.m[o];
    p[i] = P.p[o];
    rr[i] = P.r[o];
    bx[i] = P.b_ext[o];
    cw[i] = P.c_out[o];
    const int slot = tid / 16 + (kWave * kScWaves / 16) * i;
    xs[slot / 4][col][slot % 4] = (float)x[i];
  }
  __syncthreads();
  const long long base = step_first(P);
  bool bad = false;
  float e = base < sl.n_exc ? P.e_ext[sl.e_off + base] : 0.f;
  for (int s0 = 0; s0 < P.n_steps; s0 += kScChunk) {
    const int js = min(kScChunk, P.n_steps - s0);
    for (int j = 0; j < js; ++j) {
      // the next step's excitation, a step ahead
      const long long nn = base + s0 + j + 1;
      const float en = nn < sl.n_exc ? P.e_ext[sl.e_off + nn] : 0.f;
      float bq[T][KS];
      v4f xd[T], F[T];
#pragma unroll
      for (int t = 0; t < T; ++t) {
#pragma unroll
        for (int s = 0; s < KS; ++s) bq[t][s] = xs[4 * (G.part[t] & 3) + s][col][quad];
        xd[t] = *reinterpret_cast<const v4f*>(xs[4 * t + quad][col]);
        F[t] = (v4f){0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        v4f V[T];
#pragma unroll
        for (int t = 0; t < T; ++t) V[t] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
          for (int t = 0; t < T; ++t) V[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(A[r][t][s], bq[t][s], V[t], 0, 0, 0);
        float eta = 0.f;
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i) eta = fmaf(V[t][i], xd[t][i], eta);
        const float es = s2[r] * quad_sum(eta);
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i) F[t][i] = fmaf(es, V[t][i], F[t][i]);
      }
#pragma unroll
      for (int t = 0; t < T; ++t) *reinterpret_cast<v4f*>(red[wave][t][lane]) = F[t];
      float yp = 0.f;
#pragma unroll
      for (int i = 0; i < NP; ++i) yp = fmaf(cw[i], (float)x[i], yp);
      yp = quad_sum(yp);
      if (quad == 0) ys[j][wave][col] = yp;
      block_lds_sync();  // every wave's partial forces; X is read
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        const int slot = tid / 16 + (kWave * kScWaves / 16) * i;
        float f[kScWaves];
#pragma unroll
        for (int w = 0; w < kScWaves; ++w) f[w] = red[w][slot / 16][(slot % 16 / 4) * 16 + col][slot % 4];
        mode_step(x[i], d[i], m[i], p[i], rr[i], fmaf(bx[i], e, -tree_sum(f)));
        const float xh = (float)x[i];
        bad |= !isfinite(xh);
        xs[slot / 4][col][slot % 4] = xh;
      }
      e = en;
      block_lds_sync();  // X of the next step; the partial forces are read
    }
    for (int i = tid; i < kScChunk * 16; i += kWave * kScWaves) {
      const int c = i / kScChunk, j = i % kScChunk;
      const int row = P.slot[blockIdx.x * 16 + c].out_row;
      if (j >= js || row < 0 || !P.y) continue;
      float v[kScWaves];
#pragma unroll
      for (int w = 0; w < kScWaves; ++w) v[w] = ys[j][w][c];
      P.y[(long long)row * P.y_stride + s0 + j] = tree_sum(v);
    }
    block_lds_sync();  // the outputs are read
  }
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    const long long o = base_o + (kWave * kScWaves / 16) * i;
    P.x[o] = x[i];
    P.d[o] = d[i];
  }
  if (__any(bad) && lane == 0) P.flags[1] = 1;
  step_done(P);
}

// Tiles with a kernel: KS K steps of the widest class (at most 4: 16 modes)
// and R rows per wave, with the A operands (4 KS R registers) leaving room
// for the rest at two waves per SIMD.
#define SC_SHAPES(X)                                                                            \
  X(1, 1) X(1, 2) X(1, 3) X(1, 4) X(1, 6) X(1, 8) X(1, 12) X(1, 16)                             \
  X(2, 1) X(2, 2) X(2, 3) X(2, 4) X(2, 5) X(2, 6) X(2, 8) X(2, 10) X(2, 12)                     \
  X(3, 1) X(3, 2) X(3, 3) X(3, 4) X(3, 5) X(3, 6) X(3, 7) X(3, 8) X(3, 10)                      \
  X(4, 1) X(4, 2) X(4, 3) X(4, 4) X(4, 5) X(4, 6) X(4, 7)

bool shared_class_shape(int ks, int rows, int& r_tile) {
  int best = 0;
#define SC_FIT(K, RR) \
  if (K == ks && RR >= rows && (!best || RR < best)) best = RR;
  SC_SHAPES(SC_FIT)
#undef SC_FIT
  r_tile = best;
  return best > 0;
}

hipError_t launch_shared_class(const ScParams& P, int ks, int r, int n_wg, hipStream_t s) {
#define SC_RUN(K, RR)                                                                                 \
  if (ks == K && r == RR) {                                                                           \
    hipLaunchKernelGGL((shared_class_kernel<K, RR>), dim3(n_wg), dim3(kWave * kScWaves), 0, s, P);    \
    return hipGetLastError();                                                                         \
  }
  SC_SHAPES(SC_RUN)
#undef SC_RUN
  return hipErrorInvalidValue;
}

}  // namespace modal
