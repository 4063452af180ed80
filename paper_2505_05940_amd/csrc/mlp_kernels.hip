// Kernel of the proposal network (a multilayer perceptron): one kernel that
// runs a phase of a step, i.e. up to four independent jobs, each the BF16
// matrix product of one layer (FP32 accumulation) or a conversion, with what
// follows from it fused into its end: bias and ReLU, the gradient of the
// squared error, the ReLU mask, the column sums for the bias gradient, and
// the Adam update of FP32 master weights (gfx950).
//
// At the sizes of this network (batch 1024, layers of 512) a product is 0.5
// GFLOP, 0.3 us of matrix time, and a launch costs 3-5 us: launches and
// memory latency bound a step.  So a step is few launches (one per layer
// forward, one per layer backward), and no operand is converted, transposed
// or staged when it is read.  Whoever produces a matrix rounds it once to
// BF16 and stores it in the order in which the matrix instruction takes it:
// a 32-row by 16-k fragment of an operand is 64 lanes x 16 bytes contiguous,
// so a wave reads it with one fully coalesced load straight into registers,
// without LDS.  A matrix read along both of its indices (activations and
// gradients along features and along the batch, weights along both sides) is
// stored twice, once in each order; both are 16-byte stores from the tile in
// LDS.  Every use of an activation, gradient or weight in a product rounds it
// to BF16, so what is stored is what the product takes; the sums that need
// FP32 (bias gradients, loss, Adam) are taken from the FP32 tile before it is
// rounded.
//
// v_mfma_f32_32x32x16_bf16: lane l supplies A[l % 32][8 (l/32) + i] and
// B[8 (l/32) + i][l % 32], i < 8, and receives
// D[8 (r/4) + 4 (l/32) + r % 4][l % 32] in accumulator r < 16.
//
// A workgroup of eight waves owns a 32 x 64 tile of the result (256 tiles for
// 1024 x 512, one per CU), or 32 x 32 where that leaves CUs idle.  K is cut
// into up to eight slices, summed in their order; a wave takes 32 x 32 of one
// slice with eight fragments of each operand in flight, so that a K of 512 is
// one memory latency, and the partial tiles meet in LDS.
//
// An epoch of 32 batches of 1024 rows through 1024 -> 4 x 512 -> 5 took
// 7.4 ms with 35 launches a step (LDS-staged products with FP32 operands,
// separate slice sums, column sums, masks and Adam); with this kernel 2.5 ms,
// ten launches of 4.9 us (a layer forward) to 15 us (the last weight
// gradients), of which a batch of 128 rows still takes 6.4 us on average.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "mlp_kernels.h"

namespace modal {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

// round-to-nearest-even FP32 -> BF16 bits
__device__ __forceinline__ unsigned short to_bf16(float f) {
  return __builtin_bit_cast(unsigned short, (__bf16)f);
}

constexpr unsigned short kOff = 0x8000;  // a ReLU output that is not positive: -0

// element (r, k), k a multiple of 4, of an operand of kt fragments a row block
__device__ __forceinline__ long long frag_at(int r, int k, int kt) {
  return ((((long long)(r >> 5) * kt + (k >> 4)) * 64 + (r & 31) + 32 * ((k >> 3) & 1)) << 3) + (k & 7);
}

// Kingma & Ba: m = b1 m + (1-b1) g; v = b2 v + (1-b2) g^2;
// p -= lr (m / (1 - b1^t)) / (sqrt(v / (1 - b2^t)) + eps)
__device__ __forceinline__ void adam(float& p, float g, float& m, float& v, float lr, float b1, float b2,
                                     float eps, float c1, float c2) {
  m = b1 * m + (1.f - b1) * g;
  v = b2 * v + (1.f - b2) * g * g;
  p -= lr * (m / c1) / (sqrtf(v / c2) + eps);
}

__device__ __forceinline__ uint4 pack8(const unsigned short* b) {
  return make_uint4(b[0] | ((unsigned)b[1] << 16), b[2] | ((unsigned)b[3] << 16), b[4] | ((unsigned)b[5] << 16),
                    b[6] | ((unsigned)b[7] << 16));
}

// four consecutive floats of a row of n, columns c .. c+3; past its end the
// row's last ones (never a branch around a load: a wait would follow it)
__device__ __forceinline__ void ld_row(const float* __restrict__ q, int c, int n, bool vec, float* v) {
  if (vec) {
    const float4 x = *reinterpret_cast<const float4*>(q + min(c, n - 4));
    v[0] = x.x, v[1] = x.y, v[2] = x.z, v[3] = x.w;
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = q[min(c + i, n - 1)];
  }
}
__device__ __forceinline__ void st_row(float* __restrict__ q, int c, int n, bool vec, const float* v) {
  if (vec) {
    *reinterpret_cast<float4*>(q + c) = make_float4(v[0], v[1], v[2], v[3]);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (c + i < n) q[c + i] = v[i];
  }
}

constexpr int kTS = 68;  // row stride of the LDS tile: 16-byte rows, no bank conflicts
constexpr int kRing = 8;  // fragments of each operand in flight per wave

// the workgroup's tile of A B^T, one partial tile per slice of K: a wave takes
// 32 x 32 of one slice at a time
__device__ __forceinline__ void product(const MlpJob& J, int m0, int n0, int n1, float (*T)[32][kTS]) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int halves = n0 + 32 < n1 ? 2 : 1;
  const uint4* A = reinterpret_cast<const uint4*>(J.A) + (long long)(m0 >> 5) * J.akt * 64 + lane;
  for (int u0 = w; u0 < J.slices * halves; u0 += kMlpThreads / 64) {
    const int z = halves == 2 ? u0 >> 1 : u0, half = halves == 2 ? u0 & 1 : 0;
    const uint4* B = reinterpret_cast<const uint4*>(J.B) + (long long)((n0 >> 5) + half) * J.bkt * 64 + lane;
    const int k0 = z * J.ks, k1 = min(J.nk, k0 + J.ks);
    v16f acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    uint4 a[kRing], b[kRing];
    // fragments past the end re-read the last one and are not multiplied
    auto get = [&](int u, int kt) {
      const int q = 64 * min(kt, k1 - 1);
      a[u] = A[q];
      b[u] = B[q];
    };
#pragma unroll
    for (int u = 0; u < kRing; ++u) get(u, k0 + u);
    for (int k = k0; k < k1; k += kRing) {
      const bool more = k + kRing < k1;
#pragma unroll
      for (int u = 0; u < kRing; ++u) {
        if (k + u < k1)
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, a[u]),
                                                        __builtin_bit_cast(v8bf, b[u]), acc, 0, 0, 0);
        if (more) get(u, k + kRing + u);
      }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r)
      T[z][8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)][32 * half + (lane & 31)] = acc[r];
  }
}

__global__ void __launch_bounds__(kMlpThreads, 4) mlp_phase(MlpPhase P) {
  __shared__ __attribute__((aligned(16))) float T[kMlpSlices][32][kTS];
  const int t = threadIdx.x;
  int blk = blockIdx.x + gridDim.x * blockIdx.y, j = 0;
#pragma unroll
  for (int i = 0; i + 1 < kMlpJobs; ++i)
    if (blk >= P.job[i].blocks && j == i) blk -= P.job[i].blocks, ++j;
  // the whole job at once: its fields come from far away, and each one that
  // is fetched where it is used adds its latency to the launch's
  const MlpJob J = P.job[j];
  if (blk >= J.blocks) return;  // (past the last row of a grid of several)
  asm volatile("" ::"s"(J.M), "s"(J.N), "s"(J.nk), "s"(J.width), "s"(J.mt), "s"(J.inv_mt), "s"(J.slices), "s"(J.ks), "s"(J.akt), "s"(J.bkt), "s"(J.mkt), "s"(J.o1kt), "s"(J.o2kt),
               "s"(J.vec), "s"(J.relu), "s"(J.A), "s"(J.B), "s"(J.src), "s"(J.idx), "s"(J.bias), "s"(J.mask),
               "s"(J.C), "s"(J.Z), "s"(J.zidx), "s"(J.p), "s"(J.m), "s"(J.v), "s"(J.o1), "s"(J.o2), "s"(J.csum),
               "s"(J.bsum), "s"(J.n_bsum), "s"(J.bg), "s"(P.loss), "s"(P.sched));
  // rows fastest: an XCD (workgroups i, i + 8, ..) keeps to its row blocks
  int tn = __umulhi(blk, J.inv_mt), tm = blk - tn * J.mt;  // tn is one too small at most
  if (tm >= J.mt) tm -= J.mt, ++tn;
  const int m0 = 32 * tm, n0 = J.width * tn, n1 = min(J.N, n0 + J.width);
  if (P.loss && blockIdx.x + blockIdx.y == 0) {  // the previous launch's partial losses, in order
    float s = 0.f;
    for (int i = t; i < P.n_lpart; i += kMlpThreads) s += P.lpart[i];
    float* red = &T[0][0][0];
    red[t] = s;
    __syncthreads();
    for (int o = kMlpThreads / 2; o > 0; o >>= 1) {
      if (t < o) red[t] += red[t + o];
      __syncthreads();
    }
    if (t == 0) *P.loss += red[0] * P.inv;
    __syncthreads();
  }
  float lr = P.lr, c1 = P.c1, c2 = P.c2;
  if (P.sched) lr = P.sched[0], c1 = P.sched[2 * P.k + 1], c2 = P.sched[2 * P.k + 2];

  // what the end of the product takes from memory, four elements a thread,
  // rows coalesced, in flight while the product runs
  const int r = t >> 4, c = 4 * (t & 15), row = m0 + r, col = n0 + c;
  const bool vec = J.vec;  // whole aligned groups of four
  float bias[4], x[4], p[4], m[4], q[4], z[4];
  ushort4 act;
  const int lrow = min(row, J.M - 1);  // loads past the end read the last row
  const long long at = (long long)lrow * J.N;
  if (J.bias) ld_row(J.bias, col, J.N, false, bias);
  if (J.mask) act = *reinterpret_cast<const ushort4*>(J.mask + frag_at(lrow, min(col, (J.N - 1) & ~3), J.mkt));
  if (J.Z) ld_row(J.Z + J.zidx[lrow] * J.N, col, J.N, false, z);
  if (J.p) {
    ld_row(J.p + at, col, J.N, vec, p);
    ld_row(J.m + at, col, J.N, vec, m);
    ld_row(J.v + at, col, J.N, vec, q);
  }
  if (J.src) ld_row(J.src + (J.idx ? J.idx[lrow] * J.N : at), col, J.N, vec, x);
  if (J.A) {
    product(J, m0, n0, n1, T);
    __syncthreads();
  }
  float sq = 0.f, v[4] = {0.f, 0.f, 0.f, 0.f};
  if (row < J.M && col < n1) {
    if (J.A) {
      float4 y[kMlpSlices];
#pragma unroll
      for (int w = 0; w < kMlpSlices; ++w)
        if (w < J.slices) y[w] = *reinterpret_cast<const float4*>(&T[w][r][c]);
#pragma unroll
      for (int w = 0; w < kMlpSlices; ++w)
        if (w < J.slices) v[0] += y[w].x, v[1] += y[w].y, v[2] += y[w].z, v[3] += y[w].w;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = x[i];
    }
    if (J.bias) {
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] += bias[i];
    }
    if (J.relu) {
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = fmaxf(v[i], 0.f);
    }
    if (J.mask) {
      if (act.x == kOff) v[0] = 0.f;
      if (act.y == kOff) v[1] = 0.f;
      if (act.z == kOff) v[2] = 0.f;
      if (act.w == kOff) v[3] = 0.f;
    }
    if (J.C) st_row(J.C + at, col, J.N, vec, v);
    if (J.Z) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (col + i < J.N) {
          const float e = v[i] - z[i];
          sq = fmaf(e, e, sq);
          v[i] = 2.f * e * P.inv;
        }
    }
    if (J.p) {
#pragma unroll
      for (int i = 0; i < 4; ++i) adam(p[i], v[i], m[i], q[i], lr, P.b1, P.b2, P.eps, c1, c2);
      st_row(J.p + at, col, J.N, vec, p);
      st_row(J.m + at, col, J.N, vec, m);
      st_row(J.v + at, col, J.N, vec, q);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = p[i];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (col + i >= J.N) v[i] = 0.f;
  }
  *reinterpret_cast<float4*>(&T[0][r][c]) = make_float4(v[0], v[1], v[2], v[3]);
  __syncthreads();

  // The tile as operand of the products to come: half of the threads take it
  // along its rows, half along its columns, with the column sums.
  const int t8 = t & 255;
  if (t < 256) {
    const int ro = t8 & 31, k = 8 * (t8 >> 5);
    if (J.o1 && n0 + k < min(16 * J.o1kt, n0 + J.width)) {
      float e[8];
      *reinterpret_cast<float4*>(e) = *reinterpret_cast<const float4*>(&T[0][ro][k]);
      *reinterpret_cast<float4*>(e + 4) = *reinterpret_cast<const float4*>(&T[0][ro][k + 4]);
      unsigned short b[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) b[i] = J.relu && !(e[i] > 0.f) ? kOff : to_bf16(e[i]);
      *reinterpret_cast<uint4*>(J.o1 + frag_at(m0 + ro, n0 + k, J.o1kt)) = pack8(b);
    }
  } else if (J.o2) {
    const int n = (t8 & 31) + 32 * (t8 >> 7), k = 8 * ((t8 >> 5) & 3);
    float e[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) e[i] = T[0][k + i][n];
    if (n0 + (n & 32) < n1) {
      unsigned short b[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) b[i] = to_bf16(e[i]);
      *reinterpret_cast<uint4*>(J.o2 + frag_at(n0 + n, m0 + k, J.o2kt)) = pack8(b);
    }
    if (J.csum) T[1][k >> 3][n] = ((e[0] + e[1]) + (e[2] + e[3])) + ((e[4] + e[5]) + (e[6] + e[7]));
  }
  if (J.csum) {
    __syncthreads();
    if (t < 64 && n0 + t < n1)
      J.csum[(long long)tm * J.N + n0 + t] = (T[1][0][t] + T[1][1][t]) + (T[1][2][t] + T[1][3][t]);
  }
  if (J.Z) {
    float* red = &T[2][0][0];
    red[t] = sq;
    __syncthreads();
    for (int o = kMlpThreads / 2; o > 0; o >>= 1) {
      if (t < o) red[t] += red[t + o];
      __syncthreads();
    }
    if (t == 0) P.lpart[blk] = red[0];
  }
  // bias gradient of the tile's rows from the row blocks' column sums,
  // sixteen threads a row
  if (J.bg && n0 == 0) {
    const int o = m0 + (t >> 4);
    float s = 0.f;
    if (o < J.M)
      for (int i = t & 15; i < J.n_bsum; i += 16) s += J.bsum[(long long)i * J.M + o];
    s += __shfl_xor(s, 1);
    s += __shfl_xor(s, 2);
    s += __shfl_xor(s, 4);
    s += __shfl_xor(s, 8);
    if (o < J.M && (t & 15) == 0) {
      J.bg[o] = s;
      if (J.p) {
        float p = J.bp[o], m = J.bm[o], q = J.bv[o];
        adam(p, s, m, q, lr, P.b1, P.b2, P.eps, c1, c2);
        J.bp[o] = p;
        J.bm[o] = m;
        J.bv[o] = q;
      }
    }
  }
}

hipError_t launch_mlp_phase(const MlpPhase& P, hipStream_t s) {
  long long n = 0;
  for (const MlpJob& j : P.job) n += j.blocks;
  // a grid's row holds less than 2^32 threads: large phases take several
  const long long x = std::min(n, 1LL << 15);
  hipLaunchKernelGGL(mlp_phase, dim3((unsigned)x, (unsigned)((n + x - 1) / x)), dim3(kMlpThreads), 0, s, P);
  return hipGetLastError();
}

}  // namespace modal
