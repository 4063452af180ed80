// Reverse sweep of small modal systems on chip (gfx950): the adjoint
// recursion of grad_kernel.hip in the layout of chip_kernel.hip, one
// workgroup of kChipWaves waves per instance with its tensor in registers.
//
// Per step, last to first, with u = r db^{n+1}, each wave forms for its rows
// V = Ht q^n and W = Ht u (the same register tile against both vectors),
// eta = V.q, w = V.u and its partial J u = 2 w V + eta W and F = eta V, which
// cross the waves through LDS behind the step's one barrier.  Every wave
// keeps the whole adjoint state and takes the same update, in FP64; of the
// five per-mode accumulators each of the first waves keeps one, and the
// per-row sums of -2 eta w stay with the wave that owns the row.  The
// recorded trajectory is staged through LDS, kChipChunk steps at a time and
// a chunk ahead, in lane order, so q^n is read from there by every wave and
// no step waits for memory.  The sweep needs more registers than the forward
// one: of a tile of more than kChipRegs floats a lane, the last columns live
// in LDS (read once a step for both vectors).
//
// Bound, like the forward kernel, by vector issue: 2 W R multiply-adds and
// two transposed row sums a wave and step, two waves per SIMD.  64 plates at
// 40/40 over 11025 steps, forward, reverse and the fit's host part: 327 ms on
// the streaming kernels, 52 here.
#include <hip/hip_runtime.h>

#include "chip_common.h"

namespace modal {

constexpr int kChipChunk = 16;  // steps staged at a time
constexpr int kChipRegs = 160;  // tensor floats per lane in registers

// columns of a tile in LDS: 0, or enough groups of four to fit the rest
__host__ __device__ constexpr int chip_lds_cols(int w, int r) {
  return w * r <= kChipRegs ? 0 : 4 * ((w * r - kChipRegs + 4 * r - 1) / (4 * r));
}
__host__ __device__ constexpr size_t chip_grad_lds(int w, int r) {
  return sizeof(float) * ((size_t)2 * kChipChunk * (kChipVec + kWave) + kChipWaves * kChipVec +
                          4 * kChipWaves * kWave + (size_t)kChipWaves * kWave * r * chip_lds_cols(w, r));
}

template <int W, int R>
__global__ void __launch_bounds__(kWave * kChipWaves) chip_grad_kernel(GradParams P) {
  constexpr int NS = kChipChunk / kChipWaves;  // staged steps per wave
  constexpr int WL = chip_lds_cols(W, R), WR = W - WL;  // columns in LDS, in registers
  static_assert(chip_grad_lds(W, R) <= 160 * 1024, "a tile whose columns do not fit the LDS");
  extern __shared__ float4 lds4[];
  float* lds = reinterpret_cast<float*>(lds4);
  // q^n of a chunk, zero past the lanes; u^n, one copy per wave; d^n of a
  // chunk; partial J u and F, by step parity; the tile's last columns
  float(*xq)[kChipChunk][kChipVec] = reinterpret_cast<float(*)[kChipChunk][kChipVec]>(lds);
  lds += 2 * kChipChunk * kChipVec;
  float(*us)[kChipVec] = reinterpret_cast<float(*)[kChipVec]>(lds);
  lds += kChipWaves * kChipVec;
  float(*dq)[kChipChunk][kWave] = reinterpret_cast<float(*)[kChipChunk][kWave]>(lds);
  lds += 2 * kChipChunk * kWave;
  float(*redJ)[kChipWaves][kWave] = reinterpret_cast<float(*)[kChipWaves][kWave]>(lds);
  lds += 2 * kChipWaves * kWave;
  float(*redF)[kChipWaves][kWave] = reinterpret_cast<float(*)[kChipWaves][kWave]>(lds);
  lds += 2 * kChipWaves * kWave;
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const ChipMap& M = P.chip[blockIdx.x];
  const UnitDev U = P.unit[M.unit];
  const InstDev I = P.inst[blockIdx.x];
  const bool vk = I.kind == KIND_VK;
  const int k = M.perm[lane];
  const int jb = M.jb[wave][lane];
  const int jl = M.jl[wave][lane];
  const long long sf = P.state_floats;
  const int so = U.state_off + max(k, 0), mo = I.mode_off + max(k, 0);

  float h[R][WR];
  float* hl = lds + (size_t)wave * kWave * R * WL + 4 * lane;  // [column group][row][lane] float4 of this wave
  chip_load<W, R>(M, I, P.H, wave, k, jb, jl, [&](int i, int t, float v) {
    if (t < WR) h[i][t] = v;
    else hl[((t - WR) / 4 * R + i) * 4 * kWave + (t - WR) % 4] = v;
  });
  for (int i = threadIdx.x; i < 2 * kChipChunk * kWave; i += kWave * kChipWaves)
    xq[i / (kChipChunk * kWave)][i / kWave % kChipChunk][kWave + i % kWave] = 0.f;
  us[wave][kWave + lane] = 0.f;

  double qb = 0., db = 0., m = 0., p = 0., r = 0., acc = 0.;
  float bx = 0.f, cw = 0.f, lam = 0.f;
  if (k >= 0) {
    qb = P.qb[so];
    db = P.db[so];
    m = P.m[mo];
    p = P.p[mo];
    r = P.r[mo];
    bx = P.b_ext[mo];
    cw = P.c_out[mo];
    lam = P.lam[mo];
    if (wave < 5) acc = P.acc[wave * sf + so];
  }
  // the row whose sums this lane gets from row_sums, if it is one of this
  // wave's; its sum over the steps of -2 eta w
  const int rl = lane < R ? M.row[wave][lane] : -1;
  double rowacc = 0.;

  // staged steps: chunk c holds steps t in [c, c + 1) kChipChunk of the sweep,
  // step t being step seg_len - 1 - t of the segment
  auto stage = [&](int c) {
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      const int j = wave + kChipWaves * i;
      const long long ro = (long long)max(P.seg_len - 1 - (c * kChipChunk + j), 0) * P.mode_floats + mo;
      xq[c & 1][j][lane] = k >= 0 ? P.rec_x[ro] : 0.f;
      dq[c & 1][j][lane] = k >= 0 ? P.rec_d[ro] : 0.f;
    }
  };
  float ybn, evn;
  auto signals = [&](int c) {  // lane j: dL/dy and the excitation of the chunk's step j
    const long long n = P.seg_base + P.seg_len - 1 - (c * kChipChunk + min(lane, kChipChunk - 1));
    const bool in = n >= P.seg_base;
    ybn = in ? P.ybar[(long long)I.out_row * P.ybar_stride + n] : 0.f;
    evn = in && n < I.n_exc ? P.e_ext[I.e_off + n] : 0.f;
  };
  const int chunks = (P.seg_len + kChipChunk - 1) / kChipChunk;
  signals(0);
  stage(0);
  __syncthreads();
  for (int c = 0; c < chunks; ++c) {
    const float yc = ybn, ec = evn;
    // the other buffer was last read in chunk c - 1, before its last barrier;
    // the barrier at this chunk's end makes it visible
    if (c + 1 < chunks) {
      signals(c + 1);
      stage(c + 1);
    }
    const int js = min(kChipChunk, P.seg_len - c * kChipChunk);
    for (int j = 0; j < js; ++j) {
      const int st = P.seg_len - 1 - (c * kChipChunk + j);  // step within the segment
      const float* X = xq[c & 1][j];
      const float yb = lane_value(yc, j), e = lane_value(ec, j);
      const double dn = fma(-p, db, qb);
      const double ud = r * dn;
      const float u = (float)ud;
      const float q = X[lane], dv = wave == 1 ? dq[c & 1][j][lane] : 0.f;
      float Ju = 0.f, F = 0.f;
      if (vk) {
        us[wave][lane] = u;
        wave_lds_sync();
        float V[R], Wv[R], eta[R], w[R];
#pragma unroll
        for (int i = 0; i < R; ++i) V[i] = Wv[i] = 0.f;
        if constexpr (W * R <= 100) {
          chip_mul<W, R>(V, h, X + jb);  // needs no u: hides its way through LDS
          chip_mul<W, R>(Wv, h, us[wave] + jb);
        } else {
          chip_mul2<W, WR, R>(V, Wv, h, hl, X + jb, us[wave] + jb);
          // W's products stay here: sunk towards their use, they would read
          // x, u and the tile's LDS part a second time
#pragma unroll
          for (int i = 0; i < R; ++i) asm volatile("" : "+v"(Wv[i]));
        }
#pragma unroll
        for (int i = 0; i < R; ++i) {
          eta[i] = V[i] * q;
          w[i] = V[i] * u;
        }
        const float es = row_sums<R>(eta, lane), ws = row_sums<R>(w, lane);
#pragma unroll
        for (int i = 0; i < R; ++i) {
          const float ei = lane_value(es, i), wi = 2.f * lane_value(ws, i);
          Ju = fmaf(V[i], wi, fmaf(Wv[i], ei, Ju));
          F = fmaf(ei, V[i], F);
        }
        rowacc -= 2.0 * (double)(es * ws);
        if (P.trec && rl >= 0) {
          float* tr = P.trec + (long long)st * 2 * P.rows_total + I.row_off + rl;
          tr[0] = es;
          tr[P.rows_total] = ws;
        }
        if (P.urec && wave == kChipWaves - 1 && k >= 0) P.urec[(long long)st * P.mode_floats + mo] = u;
        redJ[j & 1][wave][lane] = Ju;
        redF[j & 1][wave][lane] = F;
        block_lds_sync();
        Ju = wave_join(redJ[j & 1], lane);
        if (wave == 2 || wave == 4) F = wave_join(redF[j & 1], lane);
      } else if (I.kind == KIND_TENSION) {
        const float lx = lam * q;
        const float S = group_sum<kWave>(lx * q) * I.kappa, T = 2.f * group_sum<kWave>(lx * u) * I.kappa;
        F = lx * S;
        Ju = lam * fmaf(u, S, q * T);
      }
      if (wave == 0) acc = fma(dn, (double)q, acc);
      else if (wave == 1) acc = fma(-dn, (double)dv, acc);
      else if (wave == 2) acc = fma(dn, (double)fmaf(bx, e, -F), acc);
      else if (wave == 3) acc = fma((double)yb, (double)q, acc);
      else if (wave == 4) acc = fma(-ud, (double)F, acc);
      qb = fma(m, dn, qb) + fma((double)yb, (double)cw, -(double)Ju);
      db = dn;
    }
    __syncthreads();
  }
  if (k >= 0) {
    if (wave == 0) {
      P.qb[so] = qb;
      P.db[so] = db;
    }
    if (wave < 5) P.acc[wave * sf + so] = acc;
  }
  if (P.racc && rl >= 0) P.racc[I.row_off + rl] += rowacc;
}

hipError_t launch_chip_grad(const GradParams& P, int w_tile, int rows, int n_wg, hipStream_t s) {
  if (!P.chip || P.Hd) return hipErrorInvalidValue;
#define CHIP_GRAD(WW, RR)                                                                             \
  if (w_tile == WW && rows == RR) {                                                                   \
    hipLaunchKernelGGL((chip_grad_kernel<WW, RR>), dim3(n_wg), dim3(kWave * kChipWaves),               \
                       chip_grad_lds(WW, RR), s, P);                                                  \
    return hipGetLastError();                                                                         \
  }
  CHIP_SHAPES(CHIP_GRAD)
#undef CHIP_GRAD
  return hipErrorInvalidValue;
}

}  // namespace modal
