// Time stepping and reverse sweep of instances without a coupling tensor
// (tension-modulated strings and plates, linear recursions), each on a group
// of L = 16, 32 or 64 lanes of one wave, M modes per lane (gfx950).
//
// Lane i of a group owns modes i, i + L, ..., i + L (M - 1); its FP64 state
// and coefficients stay in registers for the launch.  A sample is two sums
// over the group (DPP within a 16-lane row, lane swaps between rows): the
// output y^n = sum_k c_k q_k^n and, for the tension force (paper: Sec. 3.1)
// F_k = kappa lambda_k q_k sum_j lambda_j q_j^2, the sum; then every mode's
// update (Sec. 3.2).  No barrier and no LDS.  Excitation samples are read a
// chunk of L steps ahead, one per lane, and outputs leave a chunk at a time,
// one per lane, so a step waits for no memory and the stores are coalesced.
//
// Bound by the step's dependent chain for a few instances (0.16 us a step)
// and by vector issue, about 40 instructions a step, for many.  4096 strings
// of 12 modes over 2205 samples take 0.35 ms, 30.5 ms on the streaming kernel,
// whose workgroups step their instances in turn with barriers and the state
// in global memory.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device_common.h"
#include "kernels.h"

namespace modal {

// REC: also checkpoints of the state and the trajectory (q and d per step,
// FP32) for the reverse sweep.
template <int L, int M, bool REC>
__global__ void __launch_bounds__(kWave) wave_step_kernel(StepParams P, int batch) {
  constexpr int NG = kWave / L;
  const int lane = threadIdx.x, sub = lane & (L - 1);
  const int b = blockIdx.x * NG + lane / L;
  const bool owner = b < batch;  // groups past the batch repeat its last instance, unseen
  const UnitDev U = P.unit[owner ? b : batch - 1];
  const InstDev I = P.inst[U.inst];
  const bool tension = I.kind == KIND_TENSION;
  const float kappa = tension ? I.kappa : 0.f;
  double x[M], d[M], m[M], p[M], r[M];
  float xh[M], bx[M], cw[M], lam[M];  // xh: x rounded to FP32
#pragma unroll
  for (int i = 0; i < M; ++i) {
    const int k = sub + L * i;
    const bool live = k < I.nt;
    const int so = U.state_off + k, mo = I.mode_off + k;
    x[i] = live ? P.x[so] : 0.;
    d[i] = live ? P.d[so] : 0.;
    m[i] = live ? P.m[mo] : 0.;
    p[i] = live ? P.p[mo] : 0.;
    r[i] = live ? P.r[mo] : 0.;
    bx[i] = live ? P.b_ext[mo] : 0.f;
    cw[i] = live ? P.c_out[mo] : 0.f;
    lam[i] = live && tension ? P.lam[mo] : 0.f;
    xh[i] = (float)x[i];
  }
  const long long base = step_first(P);
  auto chunk = [&](long long n0) {
    const long long t = n0 + sub;
    return t < I.n_exc ? P.e_ext[I.e_off + t] : 0.f;
  };
  const bool any_tension = __any(tension);
  float en = chunk(base);
  bool bad = false;
  int to_ckpt = 0;  // steps to the next checkpoint
  if (REC && P.ckpt) to_ckpt = (int)((P.ckpt_every - base % P.ckpt_every) % P.ckpt_every);
  for (int s0 = 0; s0 < P.n_steps; s0 += L) {
    const float ec = en;
    const bool driven = __any(base + s0 < I.n_exc);
    en = chunk(base + s0 + L);
    const int js = min(L, P.n_steps - s0);
    float yc = 0.f;  // lane j: the output of step s0 + j
    for (int j = 0; j < js; ++j) {
      if constexpr (REC) {
        const long long n = base + s0 + j;
        if (P.rec_x && owner) {
          const long long ro = (n - P.rec_base) * P.mode_floats + I.mode_off;
#pragma unroll
          for (int i = 0; i < M; ++i) {
            const int k = sub + L * i;
            if (k < I.ntp) {
              P.rec_x[ro + k] = xh[i];
              P.rec_d[ro + k] = (float)d[i];
            }
          }
        }
        if (P.ckpt) {
          if (to_ckpt == 0) {
            double* cp = P.ckpt + (n / P.ckpt_every) * 2LL * P.mode_floats + I.mode_off;
#pragma unroll
            for (int i = 0; i < M; ++i) {
              const int k = sub + L * i;
              if (k < I.ntp && owner) {
                cp[k] = x[i];
                cp[P.mode_floats + k] = d[i];
              }
            }
            to_ckpt = P.ckpt_every;
          }
          --to_ckpt;
        }
      }
      float yp = 0.f, sp = 0.f;
#pragma unroll
      for (int i = 0; i < M; ++i) {
        yp = fmaf(cw[i], xh[i], yp);
        sp = fmaf(lam[i] * xh[i], xh[i], sp);
      }
      float S = 0.f;
      if (any_tension) S = group_sum<L>(sp) * kappa;
      const float yv = group_sum<L>(yp);
      yc = sub == j ? yv : yc;
      const float e = driven ? group_lane<L>(ec, j) : 0.f;
#pragma unroll
      for (int i = 0; i < M; ++i) {
        const float F = lam[i] * xh[i] * S;
        mode_step(x[i], d[i], m[i], p[i], r[i], fmaf(bx[i], e, -F));
        xh[i] = (float)x[i];
        bad |= !isfinite(xh[i]);
      }
    }
    if (P.y && owner && sub < js) P.y[(long long)I.out_row * P.y_stride + s0 + sub] = yc;
  }
#pragma unroll
  for (int i = 0; i < M; ++i) {
    const int k = sub + L * i;
    if (owner && k < I.nt) {
      P.x[U.state_off + k] = x[i];
      P.d[U.state_off + k] = d[i];
    }
  }
  if (__any(bad) && lane == 0) P.flags[1] = 1;
  step_done(P);
}

// Reverse sweep of a recorded segment, last step first (the recursion of
// grad_kernel.hip): with u = r db,
//   F = kappa lam q S,  J u = kappa lam (u S + q T),
//   S = sum lam q^2,    T = 2 sum lam q u.
// The adjoint state and the five accumulators of a mode stay in registers;
// the record is read C steps ahead, since a step is far shorter than a load.
template <int L, int M>
__global__ void __launch_bounds__(kWave) wave_grad_kernel(GradParams P, int batch) {
  constexpr int NG = kWave / L;
  constexpr int C = M <= 2 ? 8 : 4;  // steps of the record in flight
  const int lane = threadIdx.x, sub = lane & (L - 1);
  const int b = blockIdx.x * NG + lane / L;
  const bool owner = b < batch;
  const UnitDev U = P.unit[owner ? b : batch - 1];
  const InstDev I = P.inst[U.inst];
  const bool tension = I.kind == KIND_TENSION;
  const float kappa = tension ? I.kappa : 0.f;
  const long long sf = P.state_floats;
  double qb[M], db[M], m[M], p[M], r[M], a[M][5];
  float bx[M], cw[M], lam[M];
#pragma unroll
  for (int i = 0; i < M; ++i) {
    const int k = sub + L * i;
    const bool live = k < I.nt;
    const int so = U.state_off + k, mo = I.mode_off + k;
    qb[i] = live ? P.qb[so] : 0.;
    db[i] = live ? P.db[so] : 0.;
    m[i] = live ? P.m[mo] : 0.;
    p[i] = live ? P.p[mo] : 0.;
    r[i] = live ? P.r[mo] : 0.;
    bx[i] = live ? P.b_ext[mo] : 0.f;
    cw[i] = live ? P.c_out[mo] : 0.f;
    lam[i] = live && tension ? P.lam[mo] : 0.f;
#pragma unroll
    for (int q = 0; q < 5; ++q) a[i][q] = live ? P.acc[q * sf + so] : 0.;
  }
  // step t of the sweep is step seg_len - 1 - t of the segment
  auto load = [&](float (&xr)[C][M], float (&dr)[C][M], float& yb, float& ev, int t0) {
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const long long ro = (long long)max(P.seg_len - 1 - (t0 + c), 0) * P.mode_floats + I.mode_off;
#pragma unroll
      for (int i = 0; i < M; ++i) {
        const int k = min(sub + L * i, I.nt - 1);
        xr[c][i] = P.rec_x[ro + k];
        dr[c][i] = P.rec_d[ro + k];
      }
    }
    const long long n = P.seg_base + P.seg_len - 1 - (t0 + min(sub, C - 1));
    const bool in = n >= P.seg_base;
    yb = in ? P.ybar[(long long)I.out_row * P.ybar_stride + n] : 0.f;
    ev = in && n < I.n_exc ? P.e_ext[I.e_off + n] : 0.f;
  };
  auto sweep = [&](float (&xr)[C][M], float (&dr)[C][M], float ybs, float evs, int t0) {
#pragma unroll
    for (int c = 0; c < C; ++c) {
      if (t0 + c < P.seg_len) {
        const float yb = group_lane<L>(ybs, c), e = group_lane<L>(evs, c);
        double dn[M];
        float u[M], sx = 0.f, su = 0.f;
#pragma unroll
        for (int i = 0; i < M; ++i) {
          dn[i] = fma(-p[i], db[i], qb[i]);
          u[i] = (float)(r[i] * dn[i]);
          const float lx = lam[i] * xr[c][i];
          sx = fmaf(lx, xr[c][i], sx);
          su = fmaf(lx, u[i], su);
        }
        const float S = group_sum<L>(sx), T = 2.f * group_sum<L>(su);
#pragma unroll
        for (int i = 0; i < M; ++i) {
          const float xv = xr[c][i], kl = kappa * lam[i];
          const float F = kl * xv * S, Ju = kl * fmaf(u[i], S, xv * T);
          a[i][0] = fma(dn[i], (double)xv, a[i][0]);
          a[i][1] = fma(-dn[i], (double)dr[c][i], a[i][1]);
          a[i][2] = fma(dn[i], (double)fmaf(bx[i], e, -F), a[i][2]);
          a[i][3] = fma((double)yb, (double)xv, a[i][3]);
          a[i][4] = fma(-(r[i] * dn[i]), (double)F, a[i][4]);
          qb[i] = fma(m[i], dn[i], qb[i]) + fma((double)yb, (double)cw[i], -(double)Ju);
          db[i] = dn[i];
        }
      }
    }
  };
  float xa[C][M], da[C][M], xb[C][M], dbf[C][M], ya, yb, ea, eb;
  load(xa, da, ya, ea, 0);
  for (int t0 = 0; t0 < P.seg_len; t0 += 2 * C) {
    load(xb, dbf, yb, eb, t0 + C);
    sweep(xa, da, ya, ea, t0);
    load(xa, da, ya, ea, t0 + 2 * C);
    sweep(xb, dbf, yb, eb, t0 + C);
  }
#pragma unroll
  for (int i = 0; i < M; ++i) {
    const int k = sub + L * i;
    if (owner && k < I.nt) {
      const int so = U.state_off + k;
      P.qb[so] = qb[i];
      P.db[so] = db[i];
#pragma unroll
      for (int q = 0; q < 5; ++q) P.acc[q * sf + so] = a[i][q];
    }
  }
}

// Lanes per instance and modes per lane for a batch whose largest instance
// has nt modes: 0 lanes if no kernel holds it.  One mode per lane on the
// fewest lanes is the shortest step (12 modes: 0.155 us on 16 lanes, 0.163 on
// 32, 0.177 on 64; 30 modes: 0.164 on 32 lanes, 0.171 on 16; 60 modes: 0.176
// on 64, 0.181 on 32).  Once the batch gives every SIMD more than one wave,
// issue counts instead, and fewer lanes with more modes each are faster
// (4096 instances of 30 modes: 0.187 us on 16 lanes, 0.204 on 32, 0.333 on
// 64; of 60 modes: 0.239, 0.247, 0.339).
void wave_shape(int nt, int batch, int cus, int& lanes, int& m) {
  lanes = m = 0;
  if (nt > kWave * kWaveMaxM) return;
  lanes = nt <= 16 ? 16 : (nt <= 32 ? 32 : 64);
  while (lanes > 16 && (long long)batch * lanes > 4LL * kWave * cus && nt <= lanes / 2 * kWaveMaxM) lanes /= 2;
  m = (nt + lanes - 1) / lanes;
}

#define WV_M(LL, CALL)                                                        \
  switch (m) {                                                                \
    case 1: CALL(LL, 1); break;                                               \
    case 2: CALL(LL, 2); break;                                               \
    case 3: CALL(LL, 3); break;                                               \
    case 4: CALL(LL, 4); break;                                               \
    default: return hipErrorInvalidValue;                                     \
  }
#define WV(CALL)                                                              \
  switch (lanes) {                                                            \
    case 16: WV_M(16, CALL) break;                                            \
    case 32: WV_M(32, CALL) break;                                            \
    case 64: WV_M(64, CALL) break;                                            \
    default: return hipErrorInvalidValue;                                     \
  }
// one unit per instance, in instance order
hipError_t launch_wave_step(const StepParams& P, int lanes, int m, int batch, hipStream_t s) {
  const int n_wg = (batch + kWave / std::max(lanes, 1) - 1) / (kWave / std::max(lanes, 1));
  if (P.ckpt || P.rec_x) {
#define WV_REC(LL, MM) hipLaunchKernelGGL((wave_step_kernel<LL, MM, true>), dim3(n_wg), dim3(kWave), 0, s, P, batch)
    WV(WV_REC)
  } else {
#define WV_RUN(LL, MM) hipLaunchKernelGGL((wave_step_kernel<LL, MM, false>), dim3(n_wg), dim3(kWave), 0, s, P, batch)
    WV(WV_RUN)
  }
  return hipGetLastError();
}
hipError_t launch_wave_grad(const GradParams& P, int lanes, int m, int batch, hipStream_t s) {
  const int n_wg = (batch + kWave / std::max(lanes, 1) - 1) / (kWave / std::max(lanes, 1));
#define WV_GRAD(LL, MM) hipLaunchKernelGGL((wave_grad_kernel<LL, MM>), dim3(n_wg), dim3(kWave), 0, s, P, batch)
  WV(WV_GRAD)
  return hipGetLastError();
}

}  // namespace modal
