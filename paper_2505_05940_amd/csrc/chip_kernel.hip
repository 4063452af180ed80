// On-chip time stepping of small modal systems (gfx950): one workgroup of
// kChipWaves waves per instance, with the instance's whole coupling tensor
// held in registers for the launch.
//
// The streaming step kernel re-reads Ht from the memory hierarchy every
// sample and, for a lone instance, spreads its rows over several workgroups
// that exchange partial forces through global memory each step; a small
// plate's step is then bound by the latency of those round trips, not by its
// arithmetic.  Here the tensor of an instance with at most 64 transverse
// modes is loaded once, laid out by the instance's ChipMap: lane p stands
// for mode perm[p], wave w keeps the in-plane rows row[w][r] (r < R), and
// for each of them lane p holds the W entries h[r][t] = Ht[n][perm[jb + t]][perm[p]]
// (t < jl, zero past it) of the one run of columns that can be nonzero
// against it: all modes for a tensor without classes; for a sine-family
// tensor, whose entries vanish unless the parity classes of the two columns
// and the row match (Sec. 5, sparsity), only the partner class, a quarter of
// them.  Per sample (paper: Sec. 3.1 modal forces, Sec. 3.2 modal update)
//   1. every wave writes q^n (rounded to FP32, lane order) to its own LDS copy;
//   2. forms, for its rows, V[n, p] = sum_t h[r][t] q[jb + t] (a wave's rows
//      share jb, so each q read serves all of them), eta_n = sum_p V[n, p] q_p
//      (row_sums) and its partial force F_p = sum_n eta_n V[n, p];
//   3. writes the partial force to LDS and, after the step's one barrier,
//      adds all waves' partials and advances its lane's mode in FP64,
//      d+ = m X - p d + r (b e - F), X+ = X + d+.
// Every wave keeps the whole state and takes the same update, to the same
// bits, so that q^n need not cross a second barrier.  The output's products
// c_k q_k^n go to LDS step by step and are summed 64 steps at a time, a step
// per lane, by the last wave; excitation samples are read 64 ahead.
// Tension-modulated instances need no tensor: each wave forms
// F_k = kappa lambda_k q_k sum_j lambda_j q_j^2 itself.  Linear instances
// have F = 0.
//
// Bound by vector issue (two waves per SIMD, W R multiply-adds a wave) and
// the latency of the LDS round trips and the barrier: a 40/40 plate by class
// (a tile of 12 columns and 5 or 6 rows) steps in 0.57 us.  With wave 0 alone
// keeping the state, a second barrier for q^n, a full wave sum per row and the
// output summed every step it took 0.84 us (0.95 with a float-float state).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "chip_common.h"

namespace modal {

// W: tensor columns held per row and lane (>= every jl, multiple of 4);
// R: rows per wave (>= every wave's row count); REC: also checkpoints of the
// state and the trajectory for the reverse sweep.
template <int W, int R, bool REC>
__global__ void __launch_bounds__(kWave * kChipWaves) chip_kernel(StepParams P) {
  constexpr int kYStride = kWave + 4;
  __shared__ __align__(16) float xs[kChipWaves][kChipVec];      // q^n, one copy per wave
  __shared__ float red[2][kChipWaves][kWave];                   // partial forces, by step parity
  __shared__ __align__(16) float ys[kWave][kYStride];           // c_k q_k^n of 64 steps
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);  // wave-uniform
  const ChipMap& M = P.chip[blockIdx.x];
  const UnitDev U = P.unit[M.unit];
  const InstDev I = P.inst[blockIdx.x];
  const bool vk = I.kind == KIND_VK;
  const int k = M.perm[lane];  // this lane's mode (-1: none)
  const int jb = M.jb[wave][lane];
  const int jl = M.jl[wave][lane];
  // the mode this lane records: its own, or for the first lanes without one
  // the zeros between nt and ntp, which a reverse sweep on the streaming
  // kernel reads with the modes (64 lanes hold nt modes and that many zeros)
  int kr = k;
  if (REC && k < 0) {
    const int idle = __popcll(__ballot(k < 0) & ((1ull << lane) - 1));
    if (idle < I.ntp - I.nt) kr = I.nt + idle;
  }

  float h[R][W];
  chip_load<W, R>(M, I, P.H, wave, k, jb, jl, [&](int i, int t, float v) { h[i][t] = v; });
  float* Xc = xs[wave];
  Xc[kWave + lane] = 0.f;

  double x = 0., d = 0., m = 0., p = 0., r = 0.;
  float bx = 0.f, cw = 0.f, lam = 0.f;
  if (k >= 0) {
    const int so = U.state_off + k, mo = I.mode_off + k;
    x = P.x[so];
    d = P.d[so];
    m = P.m[mo];
    p = P.p[mo];
    r = P.r[mo];
    bx = P.b_ext[mo];
    cw = P.c_out[mo];
    lam = P.lam[mo];
  }
  // every wave has its copy of the state before the first one to finish writes
  // it back (steps of an instance without a tensor have no barrier)
  __syncthreads();
  float xh = (float)x;
  const long long base = step_first(P);
  auto chunk = [&](long long n0) {
    const long long t = n0 + lane;
    return t < I.n_exc ? P.e_ext[I.e_off + t] : 0.f;
  };
  float en = chunk(base);
  bool bad = false;
  int to_ckpt = 0;  // steps to the next checkpoint
  if (REC && P.ckpt) to_ckpt = (int)((P.ckpt_every - base % P.ckpt_every) % P.ckpt_every);
  for (int s0 = 0; s0 < P.n_steps; s0 += kWave) {
    const float ec = en;
    const bool driven = base + s0 < I.n_exc;
    en = chunk(base + s0 + kWave);
    const int js = min(kWave, P.n_steps - s0);
    for (int j = 0; j < js; ++j) {
      Xc[lane] = xh;
      if (wave == kChipWaves - 1) ys[j][lane] = cw * xh;
      if constexpr (REC) {
        const long long n = base + s0 + j;
        if (wave == kChipWaves - 2 && P.rec_x && kr >= 0) {
          const long long ro = (n - P.rec_base) * P.mode_floats + I.mode_off + kr;
          P.rec_x[ro] = xh;
          P.rec_d[ro] = (float)d;
        }
        if (P.ckpt) {
          if (to_ckpt == 0) {
            if (wave == kChipWaves - 2 && kr >= 0) {
              double* cp = P.ckpt + (n / P.ckpt_every) * 2LL * P.mode_floats + I.mode_off + kr;
              cp[0] = x;
              cp[P.mode_floats] = d;
            }
            to_ckpt = P.ckpt_every;
          }
          --to_ckpt;
        }
      }
      float F = 0.f;
      if (vk) {
        wave_lds_sync();
        float V[R], eta[R];
#pragma unroll
        for (int i = 0; i < R; ++i) V[i] = 0.f;
        chip_mul<W, R>(V, h, Xc + jb);
#pragma unroll
        for (int i = 0; i < R; ++i) eta[i] = V[i] * xh;
        const float es = row_sums<R>(eta, lane);
#pragma unroll
        for (int i = 0; i < R; ++i) F = fmaf(lane_value(es, i), V[i], F);
        red[j & 1][wave][lane] = F;
        block_lds_sync();  // every wave's partial force
        F = wave_join(red[j & 1], lane);
      } else if (I.kind == KIND_TENSION) {
        const float S = group_sum<kWave>(lam * xh * xh) * I.kappa;
        F = lam * xh * S;
      }
      const float e = driven ? lane_value(ec, j) : 0.f;
      mode_step(x, d, m, p, r, fmaf(bx, e, -F));
      xh = (float)x;
      bad |= !isfinite(xh);
    }
    if (wave == kChipWaves - 1) {
      wave_lds_sync();
      // as a tree, so that 64 modes cost six roundings; in loops, which leave
      // the tile its registers
      float4 a = f4(0.f);
#pragma unroll 1
      for (int i = 0; i < kWave; i += 32) {
        float4 t = f4(0.f);
#pragma unroll 1
        for (int g = i; g < i + 32; g += 16) {
          const float* q = &ys[lane][g];
          float4 u = ld4(q);
          u = add4(u, ld4(q + 4));
          asm volatile("" : "+v"(u.x), "+v"(u.y), "+v"(u.z), "+v"(u.w));
          t = add4(t, add4(u, add4(ld4(q + 8), ld4(q + 12))));
        }
        a = add4(a, t);
      }
      if (lane < js && P.y) P.y[(long long)I.out_row * P.y_stride + s0 + lane] = (a.x + a.y) + (a.z + a.w);
      wave_lds_sync();
    }
  }
  if (wave == 0) {
    if (k >= 0) {
      const int so = U.state_off + k;
      P.x[so] = x;
      P.d[so] = d;
    }
    if (__any(bad) && lane == 0) P.flags[1] = 1;
    step_done(P);
  }
}

// The smallest tile with a kernel that holds max_w columns and max_rows rows
// per wave.
bool chip_shape(int max_w, int max_rows, int& w_tile, int& rows) {
  int w = 0, r = 0;
  long best = -1;
#define CHIP_FIT(WW, RR)                                                       \
  if (WW >= max_w && RR >= max_rows && (best < 0 || WW * RR < best)) {         \
    best = WW * RR;                                                            \
    w = WW;                                                                    \
    r = RR;                                                                    \
  }
  CHIP_SHAPES(CHIP_FIT)
#undef CHIP_FIT
  if (best < 0 || best > kChipTile) return false;
  w_tile = w;
  rows = r;
  return true;
}

hipError_t launch_chip(const StepParams& P, int w_tile, int rows, int n_wg, hipStream_t s) {
  if (!P.chip) return hipErrorInvalidValue;
  const bool rec = P.ckpt || P.rec_x;
#define CHIP_RUN(WW, RR)                                                                                \
  if (w_tile == WW && rows == RR) {                                                                     \
    if (rec)                                                                                            \
      hipLaunchKernelGGL((chip_kernel<WW, RR, true>), dim3(n_wg), dim3(kWave * kChipWaves), 0, s, P);   \
    else                                                                                                \
      hipLaunchKernelGGL((chip_kernel<WW, RR, false>), dim3(n_wg), dim3(kWave * kChipWaves), 0, s, P);  \
    return hipGetLastError();                                                                           \
  }
  CHIP_SHAPES(CHIP_RUN)
#undef CHIP_RUN
  return hipErrorInvalidValue;
}

}  // namespace modal
