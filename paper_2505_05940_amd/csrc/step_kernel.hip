// Persistent time-stepping kernel for batches of modal systems (gfx950).
//
// A workgroup (one, four or eight 64-lane waves) owns a fixed list of work units
// for the whole launch; a unit is either a whole instance or a slab of
// in-plane rows of a von Karman instance whose coupling tensor is split over
// several workgroups; the waves of a workgroup share a unit's rows.  Per audio sample (paper: Sec. 3.2, modal oscillator
// update) each unit
//   1. publishes q^n (rounded to FP32) to LDS and writes the output sample
//      y^n = sum_k c_k q_k^n (modal-to-physical transform at one point),
//   2. evaluates its share of the nonlinear modal force (Sec. 3.1):
//        von Karman, one pass over its rows of Ht:  V[n,k] = sum_j Ht[n][j][k] q_j
//        (Ht symmetric in its last two indices), eta_n = sum_k V[n,k] q_k,
//        F_k += eta_n V[n,k];
//        tension-modulated: F_k = kappa lambda_k q_k sum_j lambda_j q_j^2,
//   3. advances the state in FP64 in increment form
//        d^{n+1} = m q^n - p d^n + r (f_ext^n - F^n),  q^{n+1} = q^n + d^{n+1}
//      (m = g + p - 1 = -r omega^2 for Stormer-Verlet), where instances split
//      over several workgroups first exchange their partial forces through
//      global memory and wait until every slab of the instance has stored
//      its arrival word for the step.
// The coupling tensor is streamed from HBM once per step with 16-byte loads
// into registers, with the non-temporal hint for a batch (each element is
// used once per step) and the default policy for a latency plan, whose
// tensors stay in the caches from step to step.  LDS holds q^n and the
// cross-lane reduction of V.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.h"
#include "device_common.h"

namespace modal {

// -------------------------------------------------------- von Karman rows
// Rows [row0, row1) of one instance's Ht.  Row n is an nt x ntp matrix
// (nc = ntp/4 float4 per stored row), read as consecutive blocks of qs
// stored rows.  A block is contiguous, so lane slot v = lane + 64 j
// (j < kSweepLoads) reads float4 number v of the block: stored row
// q0 + v / nc, columns 4 (v % nc) .. +3; one sweep is a fully coalesced
// 4 KB read per wave.  Each block gets a buffer resource sized to the block,
// so idle slots (v >= qs nc) and the missing rows of the last block read
// zeros without touching memory.  Blocks are software-pipelined across rows:
// the loads of the next block are issued before the current one is used.
// At the end of a row the slot accumulators are reduced over the qs
// sub-rows through LDS (double buffered by row parity) into V[n, :] on the
// lanes owning each float4 column group (k4 = lane + 64 g), and eta_n and
// the force follow: F += eta_n V[n, :].  DEPTH buffers (2 or 3) keep
// DEPTH - 1 blocks' loads in flight; three serve small latency-bound units
// whose rows are only a block or two long.
template <int GM, int DEPTH, int POL>
__device__ void vk_rows(const float* __restrict__ Hb, int nt, int ntp, int qs, int row0,
                        int row1, const float* Xs, float* red, float4 (&Fa)[GM], int G,
                        int lane) {
  constexpr int J = kSweepLoads;
  if (row1 <= row0) return;
  const int nc = ntp >> 2;
  const int qsnc = qs * nc;
  int voff[J], sub[J];
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int v = lane + kWave * j;
    voff[j] = 16 * v;
    sub[j] = v < qsnc ? v / nc : 0;
  }
  const int nblk = (nt + qs - 1) / qs;
  const long long blk_floats = (long long)qs * ntp;
  const long long row_floats = (long long)nt * ntp;
  const int blk_bytes = 4 * qs * ntp;
  const int last_bytes = 4 * (nt - (nblk - 1) * qs) * ntp;
  // position of the block being loaded ahead; past the last row the
  // resource covers zero bytes, so the (unconditional) loads return zeros
  // without a memory access and the loop keeps a single straight-line path
  int ln = row0, lb = 0;
  auto load = [&](float4 (&h)[J]) {
    const bool live = ln < row1;
    const float* bp = Hb + (live ? (long long)ln * row_floats + (long long)lb * blk_floats : 0);
    const int bytes = live ? (lb == nblk - 1 ? last_bytes : blk_bytes) : 0;
    const v4i r = buf_rsrc(bp, bytes);
#pragma unroll
    for (int j = 0; j < J; ++j) h[j] = buf_ld4<POL>(r, voff[j]);
    if (++lb == nblk) {
      lb = 0;
      ++ln;
    }
  };
  float4 ha[J], hb[J], acc[J];
#pragma unroll
  for (int j = 0; j < J; ++j) acc[j] = f4(0.f);
  int n = row0, b = 0;
  // Uses block `hc` (row n, block b) after issuing the loads of the next
  // block into `hn`; returns false after the last row.  Two buffers used in
  // turn keep the next block's loads in flight while the current one is
  // consumed.
  auto step = [&](float4 (&hc)[J], float4 (&hn)[J]) -> bool {
    load(hn);
    const int q0 = b * qs;
#pragma unroll
    for (int j = 0; j < J; ++j) acc[j] = fma4(hc[j], Xs[min(q0 + sub[j], nt - 1)], acc[j]);
    if (++b < nblk) return true;
    // row n complete: reduce over sub-rows, then eta_n and the force
    float* rb = red + (n & 1) * qs * ntp;
#pragma unroll
    for (int j = 0; j < J; ++j)
      if (voff[j] < blk_bytes) st4(rb + (voff[j] >> 2), acc[j]);
    wave_lds_sync();
    float eta = 0.f;
    float4 V[GM];
#pragma unroll
    for (int g = 0; g < GM; ++g) {
      V[g] = f4(0.f);
      const int k4 = lane + kWave * g;
      if (g < G && k4 < nc) {
        const float4 s = sum_strided4(rb + 4 * k4, qs, ntp);
        V[g] = s;
        eta += dot4(s, ld4(Xs + 4 * k4));
      }
    }
    eta = wave_sum(eta);
#pragma unroll
    for (int g = 0; g < GM; ++g) Fa[g] = fma4(V[g], eta, Fa[g]);
#pragma unroll
    for (int j = 0; j < J; ++j) acc[j] = f4(0.f);
    b = 0;
    return ++n < row1;
  };
  load(ha);
  if (DEPTH == 2) {
    while (step(ha, hb) && step(hb, ha)) {
    }
  } else {
    float4 hx[J];
    load(hb);
    while (step(ha, hx) && step(hb, ha) && step(hx, hb)) {
    }
  }
}

// The dense sweep over a range of row blocks instead of whole rows: blocks
// [t0, t1) of the unit whose rows start at row0, block t being block t % nblk
// of row row0 + t / nblk.  Used when a workgroup owns a single unit and its
// waves share the unit's blocks evenly, so that a unit of fewer rows than
// waves keeps every wave busy.  A row that lies wholly in the range is
// finished here (eta_n V_n added to the force).  A row that the range cuts
// (at most its first and its last) gives only partial V and eta_n, which
// are linear in the blocks summed: the partial V is parked in `defer` (two
// slots of ntp floats) and the partial eta_n and the row index in the
// wave's exchange words (slot 0: a row the range enters mid-row, slot 1: a
// row it leaves mid-row; row -1 = unused), for vk_rows_finish.
template <int GM, int DEPTH, int POL>
__device__ void vk_rows_range(const float* __restrict__ Hb, int nt, int ntp, int qs, int row0, int t0,
                              int t1, const float* Xs, float* red, float4 (&Fa)[GM], int G, int lane,
                              float* defer, float* xv, int* xr) {
  constexpr int J = kSweepLoads;
  if (lane == 0) {
    xr[0] = -1;
    xr[1] = -1;
  }
  if (t1 <= t0) return;
  const int nc = ntp >> 2;
  const int qsnc = qs * nc;
  int voff[J], sub[J];
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int v = lane + kWave * j;
    voff[j] = 16 * v;
    sub[j] = v < qsnc ? v / nc : 0;
  }
  const int nblk = (nt + qs - 1) / qs;
  const long long blk_floats = (long long)qs * ntp;
  const long long row_floats = (long long)nt * ntp;
  const int blk_bytes = 4 * qs * ntp;
  const int last_bytes = 4 * (nt - (nblk - 1) * qs) * ntp;
  // loader: block lt (flattened), row ln, block lb of that row
  int lt = t0, ln = row0 + t0 / nblk, lb = t0 % nblk;
  auto load = [&](float4 (&h)[J]) {
    const bool live = lt < t1;
    const float* bp = Hb + (live ? (long long)ln * row_floats + (long long)lb * blk_floats : 0);
    const int bytes = live ? (lb == nblk - 1 ? last_bytes : blk_bytes) : 0;
    const v4i r = buf_rsrc(bp, bytes);
#pragma unroll
    for (int j = 0; j < J; ++j) h[j] = buf_ld4<POL>(r, voff[j]);
    ++lt;
    if (++lb == nblk) {
      lb = 0;
      ++ln;
    }
  };
  float4 ha[J], hb[J], acc[J];
#pragma unroll
  for (int j = 0; j < J; ++j) acc[j] = f4(0.f);
  int t = t0, n = row0 + t0 / nblk, b = t0 % nblk, bfirst = b;
  auto step = [&](float4 (&hc)[J], float4 (&hn)[J]) -> bool {
    load(hn);
    const int q0 = b * qs;
#pragma unroll
    for (int j = 0; j < J; ++j) acc[j] = fma4(hc[j], Xs[min(q0 + sub[j], nt - 1)], acc[j]);
    ++t;
    if (++b < nblk && t < t1) return true;
    // the row, or the range's share of it, is summed
    float* rb = red + (n & 1) * qs * ntp;
#pragma unroll
    for (int j = 0; j < J; ++j)
      if (voff[j] < blk_bytes) st4(rb + (voff[j] >> 2), acc[j]);
    wave_lds_sync();
    float eta = 0.f;
    float4 V[GM];
#pragma unroll
    for (int g = 0; g < GM; ++g) {
      V[g] = f4(0.f);
      const int k4 = lane + kWave * g;
      if (g < G && k4 < nc) {
        const float4 sv = sum_strided4(rb + 4 * k4, qs, ntp);
        V[g] = sv;
        eta += dot4(sv, ld4(Xs + 4 * k4));
      }
    }
    eta = wave_sum(eta);
    if (bfirst == 0 && b == nblk) {
#pragma unroll
      for (int g = 0; g < GM; ++g) Fa[g] = fma4(V[g], eta, Fa[g]);
    } else {
      const int slot = bfirst > 0 ? 0 : 1;
#pragma unroll
      for (int g = 0; g < GM; ++g) {
        const int k4 = lane + kWave * g;
        if (g < G && k4 < nc) st4(defer + slot * ntp + 4 * k4, V[g]);
      }
      if (lane == 0) {
        xv[slot] = eta;
        xr[slot] = n;
      }
    }
#pragma unroll
    for (int j = 0; j < J; ++j) acc[j] = f4(0.f);
    b = 0;
    bfirst = 0;
    ++n;
    return t < t1;
  };
  load(ha);
  if (DEPTH == 2) {
    while (step(ha, hb) && step(hb, ha)) {
    }
  } else {
    float4 hx[J];
    load(hb);
    while (step(ha, hx) && step(hb, ha) && step(hx, hb)) {
    }
  }
}

// Completes the rows that vk_rows_range left to several waves, after a
// workgroup barrier: eta_n is the sum of the partials of every wave that
// holds row n, and each of those waves adds eta_n times its
// partial V_n.  xv, xr: the exchange words of all nw waves (this wave's at
// 2 wave).
template <int GM>
__device__ void vk_rows_finish(const float* xv, const int* xr, int nw, int wave, int ntp,
                               const float* defer, float4 (&Fa)[GM], int G, int lane) {
  const int nc = ntp >> 2;
  // the 2 nw <= 16 words, one a lane of each row of 16 lanes (read in turn by
  // every lane they cost 1 us of a 100/100 plate's step)
  const int i = lane & 15;
  const int ri = i < 2 * nw ? xr[i] : -1;
  const float vi = i < 2 * nw ? xv[i] : 0.f;
#pragma unroll
  for (int slot = 0; slot < 2; ++slot) {
    const int n = xr[2 * wave + slot];
    const float eta = group_sum<16>(ri == n ? vi : 0.f);
    if (n < 0) continue;
#pragma unroll
    for (int g = 0; g < GM; ++g) {
      const int k4 = lane + kWave * g;
      if (g < G && k4 < nc) Fa[g] = fma4(ld4(defer + slot * ntp + 4 * k4), eta, Fa[g]);
    }
  }
}

// ---------------------------------------------- parity-blocked von Karman rows
// Rows [row0, row1) of an instance stored parity-blocked: modes are grouped
// by class (class i on internal modes [cls[i], cls[i+1])), and in-plane row
// n holds, per class i, the rows of class i against the columns of class
// j = jmap[n][i] only (every other entry of those rows is zero), as a block
// as wide as class j (padded to 4) at its own offset (the second int4 of the
// row's map entry).  The sweep is the dense one applied to each (n, i) block
// in turn: pieces of qs = min(rows, 256 / (width / 4)) stored rows (at most 64 of
// a block that stands for its transpose, whose row sums are one a lane), lane slot
// v = lane + 64 j reading float4 v of the piece (sub-row v / (width / 4)),
// buffer resources sized to the valid rows, the next piece's loads issued
// before the current one is used.  Accumulating along the
// stored rows of block (n, i) gives V[n, k] for the modes k of class j
// (Ht symmetric), so at the end of each block the slot accumulators are
// reduced over the qs sub-rows through LDS onto the lanes owning those
// modes; at the end of row n, eta_n and the force follow as in the dense
// sweep.  The loader walks (n, i, block) one block ahead of the arithmetic
// and hands each block's target range and end-of-class/row flags along;
// each block's loads are issued before the previous one is used.
// When an in-plane row's blocks come in transposed pairs ((i, j) and (j, i),
// i != j) only (i, j) is stored (jmap entry j | 8): its stored rows also
// give V for class i by row dot products with q over class j, reduced over
// each row's float4 groups through LDS and collected per row in an LDS
// vector (vrow) that joins V at the end of the in-plane row.
struct BlkMeta {
  int q0;     // first stored row (internal mode) of the block
  int tc;     // first float4 column group of the target class
  int tlen;   // float4 column groups of the target class
  int flags;  // 1: last block of its class, 2: last of its row, 4: last overall,
              // 8: the block also stands for its transpose (row dot products)
  int rows;   // valid stored rows in the block
  int qs;     // sub-rows of the block's slot layout (256 / tlen, at most the class; 64 if flag 8)
};

__device__ __forceinline__ int sel4(const int4 v, int i) {
  return i == 0 ? v.x : (i == 1 ? v.y : (i == 2 ? v.z : v.w));
}

template <int GM>
__device__ void vk_rows_blk(const float* __restrict__ Hb, const int4* __restrict__ jm,
                            const InstDev& I, int row0, int row1, const float* Xs,
                            float* red, float4 (&Fa)[GM], int G, int lane) {
  constexpr int J = kSweepLoads;
  constexpr int kSlotFloats = 4 * J * kWave;  // floats of one piece's slot layout
  if (row1 <= row0) return;
  const int ntp = I.ntp;
  const int nc_modes = ntp >> 2;
  // class boundaries (a private array; read through selects instead, it left
  // scratch but measured 9 % slower on the 256-plate batch)
  int cb[5];
#pragma unroll
  for (int i = 0; i < 5; ++i) cb[i] = I.cls[i];
  auto co = [&](int i) { return cb[i]; };
  // one piece's slot layout for the class-end reductions (a wave's LDS
  // operations complete in order, so one buffer serves them all)
  float* rd = red + kSlotFloats;  // [kSweepLoads * 64] per-slot row dot partials
  float* vrow = rd + J * kWave;       // [ntp] row-dot part of V for the current row
  for (int k = lane; k < ntp; k += kWave) vrow[k] = 0.f;
  // loader position: row ln, class li, piece lb; jv, jo = map entries and
  // block offsets of row ln
  int ln = row0, li = 0, lb = 0;
  int4 jv = jm[2 * row0], jo = jm[2 * row0 + 1];
  auto has_block = [&](int i) { return co(i + 1) > co(i) && sel4(jv, i) >= 0; };
  // a paired block's partner (-1) is skipped like an empty one
  auto next_row = [&]() {
    if (++ln < row1) {
      jv = jm[2 * ln];
      jo = jm[2 * ln + 1];
    }
  };
  auto to_data = [&]() {  // first (row, class) at or after (ln, li) with a block
    while (ln < row1) {
      while (li < 4 && !has_block(li)) ++li;
      if (li < 4) return;
      next_row();
      li = 0;
    }
  };
  to_data();
  if (ln >= row1) return;  // no stored block in these rows
  auto load = [&](float4 (&h)[J], BlkMeta& m) {
    const bool live = ln < row1;
    const float* bp = Hb;
    int bytes = 0;
    m = BlkMeta{0, 0, 0, 0, 0, 1};
    if (live) {
      const int R = co(li + 1) - co(li);
      const int je = sel4(jv, li);
      const int tj = je & 7;
      m.tc = co(tj) >> 2;
      m.tlen = (co(tj + 1) - co(tj)) >> 2;
      m.qs = (je >> 4) & 511;  // from the map entry
      const int nb = je >> 13;  // pieces of the block
      m.q0 = co(li) + lb * m.qs;
      m.rows = min(m.qs, R - lb * m.qs);
      bp = Hb + sel4(jo, li) + (long long)lb * m.qs * 4 * m.tlen;
      bytes = 16 * m.rows * m.tlen;
      if (je & 8) m.flags = 8;
      if (++lb == nb) {
        m.flags |= 1;
        lb = 0;
        ++li;
        while (li < 4 && !has_block(li)) ++li;
        if (li == 4) {
          m.flags |= 2;
          li = 0;
          next_row();
          to_data();
          if (ln >= row1) m.flags |= 4;
        }
      }
    }
    const v4i r = buf_rsrc(bp, bytes);
#pragma unroll
    for (int j = 0; j < J; ++j) h[j] = buf_ld4(r, 16 * (lane + kWave * j));
  };
  float4 ha[J], hb[J], acc[J], V[GM];
  BlkMeta ma, mb;
#pragma unroll
  for (int j = 0; j < J; ++j) acc[j] = f4(0.f);
#pragma unroll
  for (int g = 0; g < GM; ++g) V[g] = f4(0.f);
  // consumes block `hc` after issuing the loads of the next block into `hn`
  auto step = [&](float4 (&hc)[J], const BlkMeta& mc, float4 (&hn)[J], BlkMeta& mn) -> bool {
    load(hn, mn);
    // sub-row of each slot in this block's layout: v / tlen (v < 256, so the
    // rounded reciprocal with half a slot of margin floors exactly)
    const float inv = __builtin_amdgcn_rcpf((float)mc.tlen);
    int sub[J];
#pragma unroll
    for (int j = 0; j < J; ++j) sub[j] = (int)(((float)(lane + kWave * j) + 0.5f) * inv);
#pragma unroll
    for (int j = 0; j < J; ++j) acc[j] = fma4(hc[j], Xs[min(mc.q0 + sub[j], ntp - 1)], acc[j]);
    if (mc.flags & 8) {
      // transposed contribution: V[q0 + t] += sum_c S[t][c] q[class j][c]
#pragma unroll
      for (int j = 0; j < J; ++j) {
        const int v = lane + kWave * j;
        const int c4 = min(v - sub[j] * mc.tlen, mc.tlen - 1);  // float4 column group of slot v
        rd[v] = dot4(hc[j], ld4(Xs + 4 * (mc.tc + c4)));
      }
      wave_lds_sync();
      if (lane < mc.rows) vrow[mc.q0 + lane] += sum_run(rd + lane * mc.tlen, mc.tlen);
    }
    if (mc.flags & 1) {
      // block row of class i done: reduce over sub-rows onto the target modes
      float* rb = red;
      const int wj = 4 * mc.tlen;
#pragma unroll
      for (int j = 0; j < J; ++j) {
        const int v = lane + kWave * j;
        if (v < mc.qs * mc.tlen) st4(rb + 4 * v, acc[j]);
      }
      wave_lds_sync();
#pragma unroll
      for (int g = 0; g < GM; ++g) {
        const int k4 = lane + kWave * g;
        const int c4 = k4 - mc.tc;
        if (g < G && c4 >= 0 && c4 < mc.tlen) {
          V[g] = add4(V[g], sum_strided4(rb + 4 * c4, mc.qs, wj));
        }
      }
#pragma unroll
      for (int j = 0; j < J; ++j) acc[j] = f4(0.f);
    }
    if (mc.flags & 2) {
      // row n done: V gets the row-dot part, then eta_n and the force
      wave_lds_sync();
      float eta = 0.f;
#pragma unroll
      for (int g = 0; g < GM; ++g) {
        const int k4 = lane + kWave * g;
        if (g < G && k4 < nc_modes) {
          V[g] = add4(V[g], ld4(vrow + 4 * k4));
          st4(vrow + 4 * k4, f4(0.f));
          eta += dot4(V[g], ld4(Xs + 4 * k4));
        }
      }
      eta = wave_sum(eta);
#pragma unroll
      for (int g = 0; g < GM; ++g) {
        Fa[g] = fma4(V[g], eta, Fa[g]);
        V[g] = f4(0.f);
      }
    }
    return !(mc.flags & 4);
  };
  load(ha, ma);
  while (step(ha, ma, hb, mb) && step(hb, mb, ha, ma)) {
  }
}

// Where one unit's state and its instance's per-mode coefficients live: in
// global memory, or resident in LDS for the whole launch.
struct ModeRefs {
  double *x, *d;
  const double *m, *p, *r;
  const float *b, *c, *lam;
};

// Per-mode state update of the float4 groups owned by this lane; e is this
// step's excitation sample.
template <int GM>
__device__ __forceinline__ void update_groups(const ModeRefs& M, int nc, float e,
                                              const float4 (&F)[GM], int G, int lane,
                                              int* flags) {
  bool bad = false;
#pragma unroll
  for (int g = 0; g < GM; ++g) {
    const int k4 = lane + kWave * g;
    if (g < G && k4 < nc) {
      const int o = 4 * k4;
      f64x4 x = ld4d(M.x + o), d = ld4d(M.d + o);
      const f64x4 m = ld4d(M.m + o), p = ld4d(M.p + o), r = ld4d(M.r + o);
      const float4 b4 = ld4(M.b + o);
      const float b[4] = {b4.x, b4.y, b4.z, b4.w}, f[4] = {F[g].x, F[g].y, F[g].z, F[g].w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        mode_step(x.v[i], d.v[i], m.v[i], p.v[i], r.v[i], fmaf(b[i], e, -f[i]));
        bad |= !isfinite((float)x.v[i]);
      }
      st4d(M.x + o, x);
      st4d(M.d + o, d);
    }
  }
  if (__any(bad) && lane == 0) atomicOr(&flags[1], 1);
}

// GM: float4 column groups per lane the launch supports (modes <= 256 GM).
// NW: waves per workgroup.  A unit's rows are divided among the NW waves,
// each sweeping its share with its own LDS reduction region; the per-wave
// partial forces are summed through those regions by wave 0, which also owns
// the output, the exchange with other workgroups and the state update.
// RES: each workgroup owns exactly one unit, whose state and coefficients
// wave 0 copies to LDS before the first step and whose state it writes back
// after the last, so that a step's output, update and recording touch no
// global memory besides the excitation sample and the output (small,
// latency-bound launches, where each global round trip is a large part of a
// step).  Only wave 0 reads or writes these arrays, so they need no barrier.
template <int GM, int NW, bool RES>
__global__ void __launch_bounds__(kWave * NW) step_kernel(StepParams P) {
  extern __shared__ float4 lds4[];
  StepLds L = step_lds(reinterpret_cast<float*>(lds4), NW, P.red_floats);
  float* Xs = L.xs;
  const int lane = threadIdx.x & (kWave - 1);
  // wave-uniform by construction; readfirstlane tells the compiler, so that
  // the row ranges and the block walks derived from it stay in scalar registers
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  float* red = L.red + wave * P.red_floats;
  const int u0 = P.wg_begin[blockIdx.x];
  const int u1 = P.wg_begin[blockIdx.x + 1];
  const long long base = step_first(P);

  auto refs = [&](const UnitDev& U, const InstDev& I) {
    ModeRefs M;
    if constexpr (RES) {
      float* R = L.res;
      const int S = P.res_stride;
      M.x = reinterpret_cast<double*>(R);
      M.d = reinterpret_cast<double*>(R + 2 * S);
      M.m = reinterpret_cast<const double*>(R + 4 * S);
      M.p = reinterpret_cast<const double*>(R + 6 * S);
      M.r = reinterpret_cast<const double*>(R + 8 * S);
      M.b = R + 10 * S;
      M.c = R + 11 * S;
      M.lam = R + 12 * S;
    } else {
      M.x = P.x + U.state_off;
      M.d = P.d + U.state_off;
      M.m = P.m + I.mode_off;
      M.p = P.p + I.mode_off;
      M.r = P.r + I.mode_off;
      M.b = P.b_ext + I.mode_off;
      M.c = P.c_out + I.mode_off;
      M.lam = P.lam + I.mode_off;
    }
    return M;
  };
  // resident state: copy in before the first step, write back after the last
  // (or when a barrier gives up); the host sizes res_stride >= ntp
  auto res_copy = [&](bool in) {
    if (!RES || wave != 0 || u1 <= u0) return;
    const UnitDev U = P.unit[u0];
    const InstDev I = P.inst[U.inst];
    const int nc = I.ntp >> 2;
    float* R = L.res;
    const int S = P.res_stride;
    double* gs[2] = {P.x + U.state_off, P.d + U.state_off};
    const double* gd[3] = {P.m + I.mode_off, P.p + I.mode_off, P.r + I.mode_off};
    const float* gc[3] = {P.b_ext + I.mode_off, P.c_out + I.mode_off, P.lam + I.mode_off};
    for (int k4 = lane; k4 < nc; k4 += kWave) {
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        double* l = reinterpret_cast<double*>(R + 2 * a * S) + 4 * k4;
        if (in)
          st4d(l, ld4d(gs[a] + 4 * k4));
        else
          st4d(gs[a] + 4 * k4, ld4d(l));
      }
      if (in) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          st4d(reinterpret_cast<double*>(R + (4 + 2 * a) * S) + 4 * k4, ld4d(gd[a] + 4 * k4));
          st4(R + (10 + a) * S + 4 * k4, ld4(gc[a] + 4 * k4));
        }
      }
    }
  };
  res_copy(true);

  for (int s = 0; s < P.n_steps; ++s) {
    const long long n = base + s;
    // ---------------- phase 1: output, force, and update of whole units
    for (int u = u0; u < u1; ++u) {
      const UnitDev U = P.unit[u];
      const InstDev I = P.inst[U.inst];
      const ModeRefs M = refs(U, I);
      const int nc = I.ntp >> 2;
      const int G = (nc + kWave - 1) / kWave;
      float spart = 0.f;
      // the excitation sample is fetched first so that its latency overlaps
      // the force evaluation
      float e = 0.f;
      if (wave == 0 && n < I.n_exc) e = P.e_ext[I.e_off + n];
      if (wave == 0) {
        float ypart = 0.f;
#pragma unroll
        for (int g = 0; g < GM; ++g) {
          const int k4 = lane + kWave * g;
          if (g < G && k4 < nc) {
            const float4 xh = to_f4(ld4d(M.x + 4 * k4));
            const float4 c = ld4(M.c + 4 * k4);
            ypart += dot4(c, xh);
            if (I.kind == KIND_VK) {
              st4(Xs + 4 * k4, xh);
            } else if (I.kind == KIND_TENSION) {
              const float4 l = ld4(M.lam + 4 * k4);
              const float4 lx = make_float4(l.x * xh.x, l.y * xh.y, l.z * xh.z, l.w * xh.w);
              spart += dot4(lx, xh);
            }
          }
        }
        if (U.slab == 0) {
          const float yv = wave_sum(ypart);
          if (lane == 0 && P.y) P.y[(long long)I.out_row * P.y_stride + s] = yv;
          if (P.ckpt && n % P.ckpt_every == 0) {
            double* cp = P.ckpt + (n / P.ckpt_every) * 2LL * P.mode_floats + I.mode_off;
            for (int g = 0; g < GM; ++g) {
              const int k4 = lane + kWave * g;
              if (g < G && k4 < nc) {
                st4d(cp + 4 * k4, ld4d(M.x + 4 * k4));
                st4d(cp + P.mode_floats + 4 * k4, ld4d(M.d + 4 * k4));
              }
            }
          }
          if (P.rec_x) {
            const long long ro = (n - P.rec_base) * P.mode_floats + I.mode_off;
            for (int g = 0; g < GM; ++g) {
              const int k4 = lane + kWave * g;
              if (g < G && k4 < nc) {
                st4(P.rec_x + ro + 4 * k4, to_f4(ld4d(M.x + 4 * k4)));
                st4(P.rec_d + ro + 4 * k4, to_f4(ld4d(M.d + 4 * k4)));
              }
            }
          }
        }
      }
      float4 Fa[GM];
#pragma unroll
      for (int g = 0; g < GM; ++g) Fa[g] = f4(0.f);
      if (I.kind == KIND_VK) {
        __syncthreads();  // q^n in LDS
        const int R = U.row1 - U.row0;
        if (RES && NW > 1 && !I.blk && 2 * R <= NW) {
          // one unit per workgroup with at most half as many rows as waves:
          // the waves share its row blocks evenly (with whole rows per wave
          // otherwise, measured faster there: 50/50 plates 9.1 us per step
          // against 11.8, 100/100 in 7-row slabs 11.7 against 14.6)
          const int nblk = (I.nt + U.qs - 1) / U.qs;
          const int T = R * nblk;
          float* xv = L.xch;
          int* xr = reinterpret_cast<int*>(L.xch + 2 * NW);
          float* defer = red + 2 * U.qs * I.ntp;
          vk_rows_range<GM, (NW == 8 && GM <= 2) ? 3 : 2, kKeep>(
              P.H + I.h_off, I.nt, I.ntp, U.qs, U.row0, (T * wave) / NW, (T * (wave + 1)) / NW, Xs, red, Fa, G,
              lane, defer, xv + 2 * wave, xr + 2 * wave);
          bool cut = false;  // a wave boundary inside a row
          for (int w = 1; w < NW; ++w) cut |= ((T * w) / NW) % nblk != 0;
          if (cut) {
            __syncthreads();  // every wave's partial eta_n of the rows it shares
            vk_rows_finish<GM>(xv, xr, NW, wave, I.ntp, defer, Fa, G, lane);
          }
        } else {
          const int r0 = U.row0 + (R * wave) / NW, r1 = U.row0 + (R * (wave + 1)) / NW;
          if (I.blk)
            vk_rows_blk<GM>(P.H + I.h_off, P.jmap + I.jmap_off, I, r0, r1, Xs, red, Fa, G, lane);
          else
            vk_rows<GM, (NW == 8 && GM <= 2) ? 3 : 2, RES ? kKeep : kStream>(
                P.H + I.h_off, I.nt, I.ntp, U.qs, r0, r1, Xs, red, Fa, G, lane);
        }
        if (NW > 1) {
#pragma unroll
          for (int g = 0; g < GM; ++g) {
            const int k4 = lane + kWave * g;
            if (g < G && k4 < nc) st4(red + 4 * k4, Fa[g]);
          }
          __syncthreads();
          if (wave == 0) {
#pragma unroll
            for (int g = 0; g < GM; ++g) {
              const int k4 = lane + kWave * g;
              if (g < G && k4 < nc)
                for (int w = 1; w < NW; ++w) Fa[g] = add4(Fa[g], ld4(L.red + w * P.red_floats + 4 * k4));
            }
          }
        }
      } else if (I.kind == KIND_TENSION && wave == 0) {
        const float S = wave_sum(spart) * I.kappa;
#pragma unroll
        for (int g = 0; g < GM; ++g) {
          const int k4 = lane + kWave * g;
          if (g < G && k4 < nc) {
            const float4 xh = to_f4(ld4d(M.x + 4 * k4));
            const float4 l = ld4(M.lam + 4 * k4);
            Fa[g] = make_float4(l.x * xh.x * S, l.y * xh.y * S, l.z * xh.z * S, l.w * xh.w * S);
          }
        }
      }
      if (wave == 0) {
        if (I.nslab == 1) {
          update_groups<GM>(M, nc, e, Fa, G, lane, P.flags);
        } else {
          // this instance's exchange region: [2][nslab][ntp] floats
          const v4i pr = buf_rsrc(P.part + I.part_off, 8 * I.nslab * I.ntp);
          const int dst = 4 * ((int)(n & 1) * I.nslab + U.slab) * I.ntp;
#pragma unroll
          for (int g = 0; g < GM; ++g) {
            const int k4 = lane + kWave * g;
            if (g < G && k4 < nc) st4_coherent(pr, dst + 16 * k4, Fa[g]);
          }
          publish_fence();
          __builtin_amdgcn_wave_barrier();
          if (lane == 0)
            __hip_atomic_store(&P.ctr[I.ctr_off + U.slab], (unsigned int)(n + 1), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        }
      }
      __syncthreads();  // LDS reused by the next unit
    }
    // ---------------- phase 2: split instances wait, sum partials, update
    for (int u = u0; u < u1; ++u) {
      const UnitDev U = P.unit[u];
      const InstDev I = P.inst[U.inst];
      if (I.nslab == 1) continue;
      if (wave == 0) {
        const bool ok = wait_slabs(P.ctr + I.ctr_off, I.nslab, (unsigned int)(n + 1), P.flags, P.timeout_ticks);
        if (lane == 0) L.flag[0] = ok ? 1 : 0;
      }
      __syncthreads();
      if (L.flag[0] == 0) {  // every wave leaves together
        res_copy(false);
        return;
      }
      const int nc = I.ntp >> 2;
      const int G = (nc + kWave - 1) / kWave;
      const v4i pr = buf_rsrc(P.part + I.part_off, 8 * I.nslab * I.ntp);
      const int src = 4 * (int)(n & 1) * I.nslab * I.ntp;  // byte offset of this step's partials
      if (RES && NW > 1 && I.nslab >= 2 * NW) {
        // one unit per workgroup and many slabs: every wave sums every NW-th
        // partial force, and wave 0 adds the waves' sums
        consume_fence();
        float4 F[GM];
#pragma unroll
        for (int g = 0; g < GM; ++g) {
          F[g] = f4(0.f);
          const int k4 = lane + kWave * g;
          if (g < G && k4 < nc) {
            F[g] = sum_slabs4_coherent(pr, src + 16 * k4, wave, NW, I.nslab, 4 * I.ntp);
            st4(red + 4 * k4, F[g]);
          }
        }
        __syncthreads();
        if (wave == 0) {
          const ModeRefs M = refs(U, I);
          float e = 0.f;
          if (n < I.n_exc) e = P.e_ext[I.e_off + n];
#pragma unroll
          for (int g = 0; g < GM; ++g) {
            const int k4 = lane + kWave * g;
            if (g < G && k4 < nc)
              for (int w = 1; w < NW; ++w) F[g] = add4(F[g], ld4(L.red + w * P.red_floats + 4 * k4));
          }
          update_groups<GM>(M, nc, e, F, G, lane, P.flags);
        }
      } else if (wave == 0) {
        consume_fence();
        const ModeRefs M = refs(U, I);
        float e = 0.f;
        if (n < I.n_exc) e = P.e_ext[I.e_off + n];
        float4 F[GM];
#pragma unroll
        for (int g = 0; g < GM; ++g) {
          F[g] = f4(0.f);
          const int k4 = lane + kWave * g;
          if (g < G && k4 < nc)
            for (int t = 0; t < I.nslab; ++t)
              F[g] = add4(F[g], ld4_coherent(pr, src + 4 * t * I.ntp + 16 * k4));
        }
        update_groups<GM>(M, nc, e, F, G, lane, P.flags);
      }
      __syncthreads();  // flag reused
    }
  }
  res_copy(false);
  step_done(P);
}

// The shared row blocks of vk_rows_range, held in registers for the launch: at
// most NB blocks of 4 KB a wave.
template <int NB>
struct RowRegs {
  float4 h[NB][kSweepLoads];
  __device__ __forceinline__ void load(const float* __restrict__ Hb, int nt, int ntp, int qs, int row0, int t0, int t1,
                                       int lane) {
    const int nblk = (nt + qs - 1) / qs;
    const int blk_bytes = 4 * qs * ntp, last_bytes = 4 * (nt - (nblk - 1) * qs) * ntp;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int t = min(t0 + i, t1 - 1), b = t % nblk;
      const v4i r = buf_rsrc(Hb + (long long)(row0 + t / nblk) * nt * ntp + (long long)b * qs * ntp,
                             t0 + i < t1 ? (b == nblk - 1 ? last_bytes : blk_bytes) : 0);
#pragma unroll
      for (int j = 0; j < kSweepLoads; ++j) h[i][j] = buf_ld4<kKeep>(r, 16 * (lane + kWave * j));
    }
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < kSweepLoads; ++j)
        asm volatile("" : "+v"(h[i][j].x), "+v"(h[i][j].y), "+v"(h[i][j].z), "+v"(h[i][j].w));
  }
  // vk_rows_range on them
  __device__ __forceinline__ void sweep(int nt, int ntp, int qs, int row0, int t0, int t1, const float* Xs, float* red,
                                        float4& Fa, int lane, float* defer, float* xv, int* xr) const {
    constexpr int J = kSweepLoads;
    if (lane == 0) {
      xr[0] = -1;
      xr[1] = -1;
    }
    if (t1 <= t0) return;
    const int nc = ntp >> 2, qsnc = qs * nc, nblk = (nt + qs - 1) / qs;
    int sub[J];
    float4 acc[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int v = lane + kWave * j;
      sub[j] = v < qsnc ? v / nc : 0;
      acc[j] = f4(0.f);
    }
    int n = row0 + t0 / nblk, b = t0 % nblk, bfirst = b;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      if (t0 + i >= t1) continue;
      const int q0 = b * qs;
#pragma unroll
      for (int j = 0; j < J; ++j) acc[j] = fma4(h[i][j], Xs[min(q0 + sub[j], nt - 1)], acc[j]);
      if (++b < nblk && t0 + i + 1 < t1) continue;
      float* rb = red + (n & 1) * qs * ntp;
#pragma unroll
      for (int j = 0; j < J; ++j)
        if (lane + kWave * j < qsnc) st4(rb + 4 * (lane + kWave * j), acc[j]);
      wave_lds_sync();
      float4 V = f4(0.f);
      float eta = 0.f;
      if (lane < nc) {
        V = sum_strided4(rb + 4 * lane, qs, ntp);
        eta = dot4(V, ld4(Xs + 4 * lane));
      }
      eta = wave_sum(eta);
      if (bfirst == 0 && b == nblk) {
        Fa = fma4(V, eta, Fa);
      } else {
        const int slot = bfirst > 0 ? 0 : 1;
        if (lane < nc) st4(defer + slot * ntp + 4 * lane, V);
        if (lane == 0) {
          xv[slot] = eta;
          xr[slot] = n;
        }
      }
#pragma unroll
      for (int j = 0; j < J; ++j) acc[j] = f4(0.f);
      b = 0;
      bfirst = 0;
      ++n;
    }
  }
  // the same for the reverse sweep (vk_rows2_range of the streaming kernel):
  // V = H q, W = H u, eta = V.q, w = V.u; J u += 2 w V + eta W, F += eta V
  __device__ __forceinline__ void sweep2(int nt, int ntp, int qs, int row0, int t0, int t1, const float* Xs,
                                         const float* Us, float* red, float4& Ju, float4& Fa, int lane, float* rrow,
                                         float* teta, float* tw, float* defer, float* xv, int* xr) const {
    constexpr int J = kSweepLoads;
    if (lane == 0) {
      xr[0] = -1;
      xr[1] = -1;
    }
    if (t1 <= t0) return;
    const int nc = ntp >> 2, qsnc = qs * nc, nblk = (nt + qs - 1) / qs, slab = qs * ntp;
    int sub[J];
    float4 aV[J], aW[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int v = lane + kWave * j;
      sub[j] = v < qsnc ? v / nc : 0;
      aV[j] = aW[j] = f4(0.f);
    }
    int n = row0 + t0 / nblk, b = t0 % nblk, bfirst = b;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      if (t0 + i >= t1) continue;
      const int q0 = b * qs;
#pragma unroll
      for (int j = 0; j < J; ++j) {
        const int qi = min(q0 + sub[j], nt - 1);
        aV[j] = fma4(h[i][j], Xs[qi], aV[j]);
        aW[j] = fma4(h[i][j], Us[qi], aW[j]);
      }
      if (++b < nblk && t0 + i + 1 < t1) continue;
#pragma unroll
      for (int j = 0; j < J; ++j)
        if (lane + kWave * j < qsnc) {
          st4(red + 4 * (lane + kWave * j), aV[j]);
          st4(red + slab + 4 * (lane + kWave * j), aW[j]);
        }
      wave_lds_sync();
      float4 V = f4(0.f), W = f4(0.f);
      float eta = 0.f, w = 0.f;
      if (lane < nc) {
        V = sum_strided4(red + 4 * lane, qs, ntp);
        W = sum_strided4(red + slab + 4 * lane, qs, ntp);
        eta = dot4(V, ld4(Xs + 4 * lane));
        w = dot4(V, ld4(Us + 4 * lane));
      }
      eta = wave_sum(eta);
      w = wave_sum(w);
      if (bfirst == 0 && b == nblk) {
        if (lane == 0) {
          if (rrow) rrow[n] = -2.f * eta * w;
          if (teta) teta[n] = eta, tw[n] = w;
        }
        Ju = fma4(V, 2.f * w, fma4(W, eta, Ju));
        Fa = fma4(V, eta, Fa);
      } else {
        const int slot = bfirst > 0 ? 0 : 1;
        if (lane < nc) {
          st4(defer + 2 * slot * ntp + 4 * lane, V);
          st4(defer + (2 * slot + 1) * ntp + 4 * lane, W);
        }
        if (lane == 0) {
          xv[2 * slot] = eta;
          xv[2 * slot + 1] = w;
          xr[slot] = n;
        }
      }
#pragma unroll
      for (int j = 0; j < J; ++j) aV[j] = aW[j] = f4(0.f);
      b = 0;
      bfirst = 0;
      ++n;
      wave_lds_sync();  // red is read before the next row's sums replace it
    }
  }
};

// ------------------------------------------------------------- latency kernel
// The step of a plan whose every workgroup owns one von Karman unit for the
// whole launch: a whole instance, or a slab of a split one, its tensor dense
// (latency plans store no blocks).  Such a plan is
// bound by the chain of one step, not by the tensor's bytes, so the chain is
// what this kernel shortens against step_kernel:
//   - a thread owns a mode (or MP), with its state and coefficients in
//     registers, instead of one wave owning four modes a lane in LDS: the sums
//     over the waves' partial forces, the update and q^n's FP32 copy are one
//     pass of all threads;
//   - slabs exchange their partial forces as 8-byte words of value and step
//     number, each stored and read whole (agent-scope atomics): what was
//     stores, a wait for them, an arrival word, a poll of all words and then
//     the reads is one store and one read, polled until its step is there
//     (every wave reads every NW-th slab, eight words a lane in flight; twelve
//     or sixteen measured slower); beyond kPairSlabs slabs each one sums a few
//     modes' words for all and publishes the sums, two such trips in all;
//   - the rows stay in registers (NB blocks of 4 KB a wave), where the slabs
//     are cut so that they fit: a 16 MB tensor is then held by 80 CUs, one of
//     32 MB by 200, and no step reads it;
//   - the output sample and the records are written while the words travel.
// Words of step n live in the half n % 2 of the region: a workgroup can only
// store step n + 2 after it has read every slab's step n + 1, which each slab
// stores after it has read step n.  A word of an older run never matches: a
// reset and a restore clear them to a step that is past.
// Lone sine plates, us a step in step_kernel and here: 66/66 10.0, 3.7;
// 100/100 8.0, 4.2; 128/128 10.2, 4.3; 160/160 13.3, 6.4; 200/200 12.0, 7.1.
// 100/100 without the rows in registers 5.3.  What is left is the exchange
// (about 2 us, two of them at 200 slabs), the reductions of a row through LDS
// and three barriers.
__device__ __forceinline__ void put_word(unsigned long long* p, unsigned int tag, float v) {
  __hip_atomic_store(p, ((unsigned long long)tag << 32) | __float_as_uint(v), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long get_word(const unsigned long long* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Every slab's partial force of the step `tag`: with up to kPairSlabs slabs each
// wave's sum over its slabs to sums[wave][stride] (to be added after a
// barrier), else the whole sum to f, thread by thread.  False if the wait was
// given up, here or elsewhere.
template <int NW, int MP>
__device__ __forceinline__ bool lat_gather(unsigned long long* words, unsigned long long* total, const InstDev& I,
                                           const UnitDev& U, unsigned int tag, float (&f)[MP], float* sums, int stride,
                                           int* flags, unsigned long long timeout) {
  constexpr int NT = kWave * NW;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), ntp = I.ntp;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const unsigned long long t0 = wall_clock64();
  bool ok = true;
  // `here`: whether this wave's words have come; else whether to go on
  auto again = [&](bool here) {
    if (__all(here)) return false;
    if (wall_clock64() - t0 > timeout)
      __hip_atomic_store(&flags[0], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    ok = __hip_atomic_load(&flags[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0;
    return ok;
  };
  if (I.nslab > kPairSlabs) {
    // each slab sums all slabs' words of its own few modes and publishes the
    // sums, which every slab then reads
    constexpr int LB = 4;  // 64-slab groups in flight
    const int seg = (ntp + I.nslab - 1) / I.nslab;
    const int k1 = min(ntp, (U.slab + 1) * seg);
    for (int k = U.slab * seg + wave; k < k1 && ok; k += NW) {
      float a = 0.f;
      for (int t = lane; t - lane < I.nslab && ok; t += LB * kWave) {
        unsigned long long v[LB];
        bool here;
        do {
          here = true;
#pragma unroll
          for (int b = 0; b < LB; ++b) v[b] = get_word(words + k * I.nslab + min(t + b * kWave, I.nslab - 1));
#pragma unroll
          for (int b = 0; b < LB; ++b) here &= (unsigned int)(v[b] >> 32) == tag;
        } while (again(here));
#pragma unroll
        for (int b = 0; b < LB; ++b)
          if (t + b * kWave < I.nslab) a += __uint_as_float((unsigned int)v[b]);
      }
      a = wave_sum(a);
      if (lane == 0 && ok) put_word(total + k, tag, a);
    }
#pragma unroll
    for (int i = 0; i < MP; ++i) {
      const int k = tid + NT * i;
      if (k - lane >= ntp || !ok) continue;
      unsigned long long v;
      do {
        v = get_word(total + min(k, ntp - 1));
      } while (again((unsigned int)(v >> 32) == tag));
      f[i] = __uint_as_float((unsigned int)v);
    }
    return ok;
  }
  constexpr int TB = 4, JB = 2;  // slabs and 64-mode groups in flight
  for (int j = 0; j < ntp; j += JB * kWave) {
    float acc[JB];
#pragma unroll
    for (int a = 0; a < JB; ++a) acc[a] = 0.f;
    for (int t = wave; t < I.nslab && ok; t += TB * NW) {
      unsigned long long v[TB][JB];
      bool here;
      do {
        here = true;
#pragma unroll
        for (int b = 0; b < TB; ++b)
#pragma unroll
          for (int a = 0; a < JB; ++a) {
            // past the end: the first slab or the last mode again
            const int tt = t + b * NW < I.nslab ? t + b * NW : t, k = min(j + a * kWave + lane, ntp - 1);
            v[b][a] = get_word(words + tt * ntp + k);
          }
#pragma unroll
        for (int b = 0; b < TB; ++b)
#pragma unroll
          for (int a = 0; a < JB; ++a) here &= (unsigned int)(v[b][a] >> 32) == tag;
      } while (again(here));
#pragma unroll
      for (int b = 0; b < TB; ++b)
        if (t + b * NW < I.nslab)
#pragma unroll
          for (int a = 0; a < JB; ++a) acc[a] += __uint_as_float((unsigned int)v[b][a]);
    }
#pragma unroll
    for (int a = 0; a < JB; ++a) {
      const int k = j + a * kWave + lane;
      if (k < ntp) sums[wave * stride + k] = acc[a];
    }
  }
  return ok;
}

template <int GM, int NW, int NB>
__global__ void __launch_bounds__(kWave * NW) lat_kernel(StepParams P) {
  extern __shared__ float4 lds4[];
  constexpr int NT = kWave * NW, MP = (4 * kWave * GM + NT - 1) / NT;
  StepLds L = step_lds(reinterpret_cast<float*>(lds4), NW, P.red_floats);
  float* Xs = L.xs;
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  float* red = L.red + wave * P.red_floats;
  const UnitDev U = P.unit[blockIdx.x];
  const InstDev I = P.inst[U.inst];
  const int ntp = I.ntp, nc = ntp >> 2, G = (nc + kWave - 1) / kWave;
  const long long base = step_first(P);
  // after the reduction regions: every wave's sum over its slabs, and its
  // share of the output sample
  float* sums = L.res;
  float* ysum = L.res + NW * P.res_stride;
  double x[MP], d[MP], m[MP], p[MP], r[MP];
  float bk[MP], ck[MP];
#pragma unroll
  for (int i = 0; i < MP; ++i) {
    const int k = min(tid + NT * i, ntp - 1);
    x[i] = P.x[U.state_off + k];
    d[i] = P.d[U.state_off + k];
    m[i] = P.m[I.mode_off + k];
    p[i] = P.p[I.mode_off + k];
    r[i] = P.r[I.mode_off + k];
    bk[i] = P.b_ext[I.mode_off + k];
    ck[i] = P.c_out[I.mode_off + k];
  }
  const int R = U.row1 - U.row0, nblk = (I.nt + U.qs - 1) / U.qs, T = R * nblk;
  const int tw0 = (T * wave) / NW, tw1 = (T * (wave + 1)) / NW;  // the wave's share of the unit's blocks
  const bool shared_rows = NB > 0 || 2 * R <= NW;
  bool cut = false;  // a wave boundary inside a row
  for (int w = 1; w < NW; ++w) cut |= ((T * w) / NW) % nblk != 0;
  float* xv = L.xch;
  int* xr = reinterpret_cast<int*>(L.xch + 2 * NW);
  float* defer = red + 2 * U.qs * ntp;
  RowRegs<NB == 0 ? 1 : NB> H;
  if (NB > 0) H.load(P.H + I.h_off, I.nt, ntp, U.qs, U.row0, tw0, tw1, lane);
  if (tid == 0) L.flag[0] = 0;
  // the state is in registers before this slab's first word goes out: with
  // every slab's words the first one may end its launch and write it back
  publish_fence();
  bool bad = false;
  int s = 0;
  for (; s < P.n_steps; ++s) {
    const long long n = base + s;
    float e = 0.f;
    if (n < I.n_exc) e = P.e_ext[I.e_off + n];
#pragma unroll
    for (int i = 0; i < MP; ++i)
      if (tid + NT * i < ntp) Xs[tid + NT * i] = (float)x[i];
    __syncthreads();
    // ---- the unit's rows, as in step_kernel
    float4 Fa[GM];
#pragma unroll
    for (int g = 0; g < GM; ++g) Fa[g] = f4(0.f);
    if (shared_rows) {
      if constexpr (NB > 0)
        H.sweep(I.nt, ntp, U.qs, U.row0, tw0, tw1, Xs, red, Fa[0], lane, defer, xv + 2 * wave, xr + 2 * wave);
      else
        vk_rows_range<GM, (NW == 8 && GM <= 2) ? 3 : 2, kKeep>(P.H + I.h_off, I.nt, ntp, U.qs, U.row0, tw0, tw1, Xs,
                                                               red, Fa, G, lane, defer, xv + 2 * wave, xr + 2 * wave);
      if (cut) {
        __syncthreads();  // every wave's partial eta_n of the rows it shares
        vk_rows_finish<GM>(xv, xr, NW, wave, ntp, defer, Fa, G, lane);
      }
    } else {
      const int r0 = U.row0 + (R * wave) / NW, r1 = U.row0 + (R * (wave + 1)) / NW;
      vk_rows<GM, (NW == 8 && GM <= 2) ? 3 : 2, kKeep>(P.H + I.h_off, I.nt, ntp, U.qs, r0, r1, Xs, red, Fa, G, lane);
    }
#pragma unroll
    for (int g = 0; g < GM; ++g) {
      const int k4 = lane + kWave * g;
      if (g < G && k4 < nc) st4(red + 4 * k4, Fa[g]);
    }
    __syncthreads();
    // ---- the unit's force, published
    const int half = (int)(n & 1);
    unsigned long long* words = P.pair + I.part_off + half * (long long)I.nslab * ntp;
    const unsigned int tag = (unsigned int)(n + 1);
    const bool owners = I.nslab > kPairSlabs;
    float f[MP];
#pragma unroll
    for (int i = 0; i < MP; ++i) {
      const int k = tid + NT * i;
      f[i] = 0.f;
      if (k < ntp) {
        for (int w = 0; w < NW; ++w) f[i] += L.red[w * P.red_floats + k];
        if (I.nslab > 1) put_word(words + (owners ? k * I.nslab + U.slab : U.slab * ntp + k), tag, f[i]);
      }
    }
    // ---- output and records of this step's state
    if (U.slab == 0) {
      float yp = 0.f;
#pragma unroll
      for (int i = 0; i < MP; ++i) {
        const int k = tid + NT * i;
        if (k >= ntp) continue;
        yp += quad_dot(ck[i], (float)x[i], lane);  // (ntp is a multiple of 4)
        if (P.ckpt && n % P.ckpt_every == 0) {
          double* cp = P.ckpt + (n / P.ckpt_every) * 2LL * P.mode_floats + I.mode_off;
          cp[k] = x[i];
          cp[P.mode_floats + k] = d[i];
        }
        if (P.rec_x) {
          const long long ro = (n - P.rec_base) * P.mode_floats + I.mode_off + k;
          P.rec_x[ro] = (float)x[i];
          P.rec_d[ro] = (float)d[i];
        }
      }
      yp = wave_sum(yp);
      if (lane == 0) ysum[wave] = yp;
    }
    // ---- every slab's force
    if (I.nslab > 1 && !lat_gather<NW, MP>(words, P.pair2 + half * P.mode_floats + I.mode_off, I, U, tag, f, sums,
                                           P.res_stride, P.flags, P.timeout_ticks) && lane == 0)
      L.flag[0] = 1;
    __syncthreads();
    if (tid == 0 && U.slab == 0 && P.y) {
      float yv[NW];
#pragma unroll
      for (int w = 0; w < NW; ++w) yv[w] = ysum[w];
#pragma unroll
      for (int h = 1; h < NW; h *= 2)
#pragma unroll
        for (int w = 0; w < NW; w += 2 * h) yv[w] += yv[w + h];  // (as wave_sum pairs the rows of a wave)
      P.y[(long long)I.out_row * P.y_stride + s] = yv[0];
    }
    if (L.flag[0]) break;  // a wait was given up; every thread leaves
    // ---- state
#pragma unroll
    for (int i = 0; i < MP; ++i) {
      const int k = tid + NT * i;
      if (k >= ntp) continue;
      if (I.nslab > 1 && !owners) {
        f[i] = 0.f;
        for (int w = 0; w < NW; ++w) f[i] += sums[w * P.res_stride + k];
      }
      mode_step(x[i], d[i], m[i], p[i], r[i], fmaf(bk[i], e, -f[i]));
      bad |= !isfinite((float)x[i]);
    }
  }
#pragma unroll
  for (int i = 0; i < MP; ++i) {
    const int k = tid + NT * i;
    if (k >= ntp || U.slab) continue;
    P.x[U.state_off + k] = x[i];
    P.d[U.state_off + k] = d[i];
  }
  if (__any(bad) && lane == 0) atomicOr(&P.flags[1], 1);
  if (s == P.n_steps) step_done(P);
}

// The reverse (adjoint) step in the same way, for the units whose rows stay in
// registers.  Only J u is exchanged: F enters the gradients alone, which are
// linear in it, so each slab sums dbar F over the steps for its own part (gs)
// and lat_sum_kernel adds the slabs.  Lone sine plates, us a step of a
// gradient less its forward pass, with grad_kernel and here: 66/66 17.8, 6.6;
// 100/100 15.0, 7.5; 128/128 18.2, 8.3; 200/200 24.5, 14.8; of a reverse sweep
// that reuses the forward run's record 5.5, 6.0, 5.8 and 8.0.  The variant of
// eight blocks spills 68 bytes a lane.
template <int NW, int NB>
__global__ void __launch_bounds__(kWave * NW) lat_grad_kernel(GradParams P) {
  extern __shared__ float4 lds4[];
  const LatGradLds L = lat_grad_lds(reinterpret_cast<float*>(lds4), NW, P.red_floats);
  float *Xs = L.xs, *Us = L.us;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), k = tid;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  float* red = L.red + wave * P.red_floats;
  const UnitDev U = P.unit[blockIdx.x];
  const InstDev I = P.inst[U.inst];
  const int ntp = I.ntp, nc = ntp >> 2;  // ntp <= 256, one mode a thread
  const bool mine = k < ntp, first = U.slab == 0;
  const int so = U.state_off + min(k, ntp - 1), mo = I.mode_off + min(k, ntp - 1);
  double qb = P.qb[so], db = P.db[so];
  const double m = P.m[mo], p = P.p[mo], r = P.r[mo];
  const float bk = P.b_ext[mo], ck = P.c_out[mo];
  double a0 = 0., a1 = 0., a2 = 0., a3 = 0., gs = 0.;
  const int R = U.row1 - U.row0, nblk = (I.nt + U.qs - 1) / U.qs, T = R * nblk;
  const int tw0 = (T * wave) / NW, tw1 = (T * (wave + 1)) / NW;
  bool cut = false;
  for (int w = 1; w < NW; ++w) cut |= ((T * w) / NW) % nblk != 0;
  float* xv = L.xch;
  int* xr = reinterpret_cast<int*>(L.xch + 4 * NW);
  float* defer = red + 2 * U.qs * ntp;
  RowRegs<NB> H;
  H.load(P.H + I.h_off, I.nt, ntp, U.qs, U.row0, tw0, tw1, lane);
  if (tid == 0) L.flag[0] = 0;
  const float* rx = P.rec_x + mo;
  const float* rd = P.rec_d + mo;
  const float* yrow = P.ybar + (long long)I.out_row * P.ybar_stride + P.seg_base;
  // a step's record is fetched a step ahead
  float xn = rx[(long long)(P.seg_len - 1) * P.mode_floats], dn_ = rd[(long long)(P.seg_len - 1) * P.mode_floats];
  float yn = yrow[P.seg_len - 1];
  for (int s = 0; s < P.seg_len; ++s) {
    const int row = P.seg_len - 1 - s;
    const long long n = P.seg_base + row, rstep = P.done_before + s;
    const float x = xn, dd = dn_, yb = yn;
    const float e = n < I.n_exc ? P.e_ext[I.e_off + n] : 0.f;
    const int next = max(row - 1, 0);
    xn = rx[(long long)next * P.mode_floats];
    dn_ = rd[(long long)next * P.mode_floats];
    yn = yrow[next];
    const double dbar = fma(-p, db, qb);  // db^{n+1}
    const float u = (float)(r * dbar);
    if (mine) {
      Xs[k] = x;
      Us[k] = u;
      if (P.urec && first) P.urec[(long long)row * P.mode_floats + mo] = u;
    }
    __syncthreads();
    float4 Ju = f4(0.f), Fa = f4(0.f);
    float* rrow = P.rrec ? P.rrec + (long long)s * P.rows_total + I.row_off : nullptr;
    float* teta = P.trec ? P.trec + row * 2LL * P.rows_total + I.row_off : nullptr;
    float* tw = teta ? teta + P.rows_total : nullptr;
    H.sweep2(I.nt, ntp, U.qs, U.row0, tw0, tw1, Xs, Us, red, Ju, Fa, lane, rrow, teta, tw, defer, xv + 4 * wave,
             xr + 2 * wave);
    if (cut) {
      __syncthreads();  // every wave's partials of the rows it shares
      const int i = lane & 15;
      const bool in = i < 2 * NW;
      const int ri = in ? xr[i] : -1;
      const float ei = in ? xv[2 * i] : 0.f, wi = in ? xv[2 * i + 1] : 0.f;
#pragma unroll
      for (int slot = 0; slot < 2; ++slot) {
        const int nr = xr[2 * wave + slot];
        const float eta = group_sum<16>(ri == nr ? ei : 0.f), w = group_sum<16>(ri == nr ? wi : 0.f);
        if (nr < 0) continue;
        if (lane < nc) {
          const float4 V = ld4(defer + 2 * slot * ntp + 4 * lane), W = ld4(defer + (2 * slot + 1) * ntp + 4 * lane);
          Ju = fma4(V, 2.f * w, fma4(W, eta, Ju));
          Fa = fma4(V, eta, Fa);
        }
        if (slot == 1 && lane == 0) {  // the wave that holds the row's first block
          if (rrow) rrow[nr] = -2.f * eta * w;
          if (teta) teta[nr] = eta, tw[nr] = w;
        }
      }
    }
    if (lane < nc) {
      st4(red + 4 * lane, Ju);
      st4(red + ntp + 4 * lane, Fa);
    }
    __syncthreads();
    const int half = (int)(rstep & 1);
    unsigned long long* words = P.pair + I.part_off + half * (long long)I.nslab * ntp;
    const unsigned int tag = (unsigned int)(rstep + 1);
    const bool owners = I.nslab > kPairSlabs;
    float ju[1] = {0.f}, f = 0.f;
    if (mine) {
      for (int w = 0; w < NW; ++w) ju[0] += L.red[w * P.red_floats + k];
      if (I.nslab > 1) put_word(words + (owners ? k * I.nslab + U.slab : U.slab * ntp + k), tag, ju[0]);
      for (int w = 0; w < NW; ++w) f += L.red[w * P.red_floats + ntp + k];
    }
    gs = fma(dbar, (double)f, gs);
    if (first) {
      a0 = fma(dbar, (double)x, a0);
      a1 = fma(-dbar, (double)dd, a1);
      a2 = fma(dbar, (double)(bk * e), a2);
      a3 = fma((double)yb, (double)x, a3);
    }
    if (I.nslab > 1 && !lat_gather<NW, 1>(words, P.pair2 + half * P.mode_floats + I.mode_off, I, U, tag, ju, L.sums,
                                          kWave * 4, P.flags, P.timeout_ticks) && lane == 0)
      L.flag[0] = 1;
    __syncthreads();
    if (L.flag[0]) return;  // a wait was given up; every thread leaves
    if (mine && I.nslab > 1 && !owners) {
      ju[0] = 0.f;
      for (int w = 0; w < NW; ++w) ju[0] += L.sums[w * kWave * 4 + k];
    }
    // qb^n = ybar c + qb^{n+1} + m db^{n+1} - (J u)
    qb = fma(m, dbar, qb) + fma((double)yb, (double)ck, -(double)ju[0]);
    db = dbar;
  }
  if (!mine) return;
  P.gs[(long long)blockIdx.x * kWave * 4 + k] += gs;
  if (first) {
    P.qb[so] = qb;
    P.db[so] = db;
    const long long sf = P.state_floats;
    P.acc[so] += a0;
    P.acc[sf + so] += a1;
    P.acc[2 * sf + so] += a2;
    P.acc[3 * sf + so] += a3;
  }
}

// Adds the slabs' sums of dbar F to the accumulators of each instance, in the
// order of the slabs.
__global__ void lat_sum_kernel(const InstDev* inst, const UnitDev* unit, int n_units, const double* gs, const double* r,
                               double* acc, int state_floats) {
  const UnitDev U = unit[blockIdx.x];
  const InstDev I = inst[U.inst];
  const int k = threadIdx.x;
  if (U.slab != 0 || k >= I.ntp) return;
  double g = 0.;
#pragma unroll 8
  for (int t = 0; t < I.nslab; ++t) g += gs[(long long)(blockIdx.x + t) * kWave * 4 + k];
  acc[2LL * state_floats + U.state_off + k] -= g;
  acc[4LL * state_floats + U.state_off + k] -= r[I.mode_off + k] * g;
}

// n words of the latency kernel's exchange, as left by the steps before
// *step_base.
__global__ void pair_fill_kernel(unsigned long long* pair, long long n, const long long* step_base) {
  const unsigned long long v = (unsigned long long)*step_base << 32;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
    pair[i] = v;
}

// Puts a context back to its initial state: the state's n doubles, n_ctr
// arrival words, n_pair exchange words, both pairs of status flags (the device's and, if there is one, the host's) and
// the step counter.
__global__ void __launch_bounds__(256) reset_kernel(double* st, const double* st0, long long n, unsigned int* ctr,
                                                    int n_ctr, unsigned long long* pair, long long n_pair,
                                                    int* dflags, int* hflags, long long* step) {
  const long long i0 = (long long)blockIdx.x * blockDim.x + threadIdx.x, di = (long long)gridDim.x * blockDim.x;
  for (long long i = i0; i < n / 2; i += di)
    reinterpret_cast<v2d*>(st)[i] = reinterpret_cast<const v2d*>(st0)[i];
  for (long long i = i0; i < n_ctr; i += di) ctr[i] = 0u;
  for (long long i = i0; i < n_pair; i += di) pair[i] = 0u;
  if (i0 < 2) {
    dflags[i0] = 0;
    if (hflags) hflags[i0] = 0;
  }
  if (i0 == 0) *step = 0;
}

__global__ void advance_kernel(long long* step_base, int n_steps) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *step_base += n_steps;
}

// Arrival words as they stand after *step_base steps from a reset: every
// slab has published every step (mod 2^32, like the waits' targets).  Lets
// a launch run on words that another context left behind.
__global__ void ctr_fill_kernel(const InstDev* inst, int batch, const long long* step_base,
                                unsigned int* ctr) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= batch) return;
  const unsigned int v = (unsigned int)(unsigned long long)*step_base;
  for (int t = 0; t < inst[b].nslab; ++t) ctr[inst[b].ctr_off + t] = v;
}

// Every slab's copy of the state from its instance's slab 0, and the arrival
// words as ctr_fill_kernel sets them: what the streaming kernel needs after
// steps on chip.
__global__ void spread_kernel(const InstDev* inst, const UnitDev* unit, int n_units, double* state, int state_floats,
                              unsigned int* ctr, const long long* step_base) {
  const UnitDev U = unit[blockIdx.x];
  const InstDev I = inst[U.inst];
  if (threadIdx.x == 0) ctr[I.ctr_off + U.slab] = (unsigned int)(unsigned long long)*step_base;
  if (U.slab == 0) return;
  int from = 0;  // the instance's slab 0
  for (int u = 0; u < n_units; ++u)
    if (unit[u].inst == U.inst && unit[u].slab == 0) from = unit[u].state_off;
  for (int k = threadIdx.x; k < I.ntp; k += blockDim.x)
    for (int a = 0; a < 2; ++a)
      state[(long long)a * state_floats + U.state_off + k] = state[(long long)a * state_floats + from + k];
}

// Symmetry and finiteness of each instance's Ht: out[2b] = max |H - H^T|,
// out[2b+1] = max |H|, both as float bits (non-negative floats order like
// their bit patterns); a non-finite entry reports +inf in both.
__global__ void check_kernel(const float* H, const InstDev* inst, int* out) {
  const InstDev I = inst[blockIdx.y];
  if (I.kind != KIND_VK || I.blk) return;  // blocked tensors are checked on the host
  const long long total = (long long)I.nin * I.nt * I.nt;
  float dmax = 0.f, hmax = 0.f;
  for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x) {
    const int j = (int)(e % I.nt);
    const long long r = e / I.nt;
    const int k = (int)(r % I.nt);
    const long long n = r / I.nt;
    const float* Hn = H + I.h_off + n * (long long)I.nt * I.ntp;
    const float a = Hn[(long long)k * I.ntp + j];
    const float b = Hn[(long long)j * I.ntp + k];
    if (!isfinite(a)) {
      dmax = INFINITY;
      hmax = INFINITY;
    } else {
      dmax = fmaxf(dmax, fabsf(a - b));
      hmax = fmaxf(hmax, fabsf(a));
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    dmax = fmaxf(dmax, __shfl_xor(dmax, o, kWave));
    hmax = fmaxf(hmax, __shfl_xor(hmax, o, kWave));
  }
  if ((threadIdx.x & (kWave - 1)) == 0) {
    atomicMax(&out[2 * blockIdx.y], __float_as_int(dmax));
    atomicMax(&out[2 * blockIdx.y + 1], __float_as_int(hmax));
  }
}

}  // namespace modal

// Launch wrappers used by the host code (same translation unit keeps the
// kernels' symbols local to this file).
namespace modal {
// gm: float4 column groups per lane needed by the widest instance (1, 2 or
// 4); nw: waves per workgroup (1, 4 or 8); P.res_stride > 0 selects the
// variant with LDS-resident state (four or eight waves, one unit per
// workgroup).
hipError_t launch_step(const StepParams& P, int gm, int nw, int n_wg, size_t lds_bytes, hipStream_t s) {
#define SL(G, W, R) hipLaunchKernelGGL((step_kernel<G, W, R>), dim3(n_wg), dim3(kWave * W), lds_bytes, s, P)
  if (P.res_stride > 0) {
    if (nw == 8) {
      if (gm <= 1) SL(1, 8, true); else if (gm <= 2) SL(2, 8, true); else SL(4, 8, true);
    } else if (nw == 4) {
      if (gm <= 1) SL(1, 4, true); else if (gm <= 2) SL(2, 4, true); else SL(4, 4, true);
    } else {
      return hipErrorInvalidValue;  // resident launches use four or eight waves
    }
  } else if (nw == 1) {
    if (gm <= 1) SL(1, 1, false); else if (gm <= 2) SL(2, 1, false); else SL(4, 1, false);
  } else if (nw == 8) {
    if (gm <= 1) SL(1, 8, false); else if (gm <= 2) SL(2, 8, false); else SL(4, 8, false);
  } else {
    if (gm <= 1) SL(1, 4, false); else if (gm <= 2) SL(2, 4, false); else SL(4, 4, false);
  }
#undef SL
  return hipGetLastError();
}
// n: even
hipError_t launch_reset(double* st, const double* st0, long long n, unsigned int* ctr, int n_ctr,
                        unsigned long long* pair, long long n_pair, int* dflags, int* hflags, long long* step,
                        hipStream_t s) {
  const long long want = (std::max({n / 2, (long long)n_ctr, n_pair}) + 255) / 256;
  hipLaunchKernelGGL(reset_kernel, dim3((unsigned)std::max<long long>(1, std::min<long long>(want, 2048))), dim3(256),
                     0, s, st, st0, n, ctr, n_ctr, pair, n_pair, dflags, hflags, step);
  return hipGetLastError();
}
hipError_t launch_advance(long long* step_base, int n, hipStream_t s) {
  hipLaunchKernelGGL(advance_kernel, dim3(1), dim3(64), 0, s, step_base, n);
  return hipGetLastError();
}
hipError_t launch_ctr_fill(const InstDev* inst, int batch, const long long* step_base, unsigned int* ctr,
                           hipStream_t s) {
  hipLaunchKernelGGL(ctr_fill_kernel, dim3((batch + 255) / 256), dim3(256), 0, s, inst, batch, step_base, ctr);
  return hipGetLastError();
}
hipError_t launch_pair_fill(unsigned long long* pair, long long n, const long long* step_base, hipStream_t s) {
  hipLaunchKernelGGL(pair_fill_kernel, dim3((unsigned)std::min<long long>((n + 255) / 256, 1024)), dim3(256), 0, s, pair,
                     n, step_base);
  return hipGetLastError();
}
hipError_t launch_spread(const InstDev* inst, const UnitDev* unit, int n_units, double* state, int state_floats,
                         unsigned int* ctr, const long long* step_base, hipStream_t s) {
  hipLaunchKernelGGL(spread_kernel, dim3(n_units), dim3(kWave), 0, s, inst, unit, n_units, state, state_floats, ctr,
                     step_base);
  return hipGetLastError();
}
// gm, nw, lds_bytes as launch_step's with resident state; nb: blocks a wave of
// the launch's units keeps in registers (0: streamed; else 4 or 8, with gm 1
// and nw 8)
hipError_t launch_lat(const StepParams& P, int gm, int nw, int nb, int n_wg, size_t lds_bytes, hipStream_t s) {
#define LL(G, W, B) hipLaunchKernelGGL((lat_kernel<G, W, B>), dim3(n_wg), dim3(kWave * W), lds_bytes, s, P)
  if (nb == 4) LL(1, 8, 4);
  else if (nb == 8) LL(1, 8, 8);
  else if (nw == 8) {
    if (gm <= 1) LL(1, 8, 0); else if (gm <= 2) LL(2, 8, 0); else LL(4, 8, 0);
  } else {
    if (gm <= 1) LL(1, 4, 0); else if (gm <= 2) LL(2, 4, 0); else LL(4, 4, 0);
  }
#undef LL
  return hipGetLastError();
}
hipError_t lat_occupancy(int* blocks_per_cu, int gm, int nw, int nb, size_t lds_bytes) {
#define LO(G, W, B) \
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, lat_kernel<G, W, B>, kWave * W, lds_bytes)
  if (nb == 4) LO(1, 8, 4);
  if (nb == 8) LO(1, 8, 8);
  if (nw == 8) {
    if (gm <= 1) LO(1, 8, 0);
    if (gm <= 2) LO(2, 8, 0);
    LO(4, 8, 0);
  }
  if (gm <= 1) LO(1, 4, 0);
  if (gm <= 2) LO(2, 4, 0);
  LO(4, 4, 0);
#undef LO
}
// nb: 4, 6 or 8
hipError_t launch_lat_grad(const GradParams& P, int nb, int n_wg, size_t lds_bytes, hipStream_t s) {
#define LG(B) hipLaunchKernelGGL((lat_grad_kernel<8, B>), dim3(n_wg), dim3(kWave * 8), lds_bytes, s, P)
  if (nb <= 4) LG(4); else if (nb <= 6) LG(6); else LG(8);
#undef LG
  return hipGetLastError();
}
hipError_t launch_lat_sum(const InstDev* inst, const UnitDev* unit, int n_units, const double* gs, const double* r,
                          double* acc, int state_floats, hipStream_t s) {
  hipLaunchKernelGGL(lat_sum_kernel, dim3(n_units), dim3(kWave * 4), 0, s, inst, unit, n_units, gs, r, acc,
                     state_floats);
  return hipGetLastError();
}
hipError_t lat_grad_occupancy(int* blocks_per_cu, int nb, size_t lds_bytes) {
#define LG(B) \
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, lat_grad_kernel<8, B>, kWave * 8, lds_bytes)
  if (nb <= 4) LG(4);
  if (nb <= 6) LG(6);
  LG(8);
#undef LG
}
hipError_t launch_check(const float* H, const InstDev* inst, int batch, int* out, hipStream_t s) {
  hipLaunchKernelGGL(check_kernel, dim3(64, batch), dim3(256), 0, s, H, inst, out);
  return hipGetLastError();
}
hipError_t step_occupancy(int* blocks_per_cu, int gm, int nw, size_t lds_bytes, bool res) {
#define SO(G, W, R) \
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, step_kernel<G, W, R>, kWave * W, lds_bytes)
  if (res) {
    if (nw == 8) {
      if (gm <= 1) SO(1, 8, true);
      if (gm <= 2) SO(2, 8, true);
      SO(4, 8, true);
    }
    if (nw == 4) {
      if (gm <= 1) SO(1, 4, true);
      if (gm <= 2) SO(2, 4, true);
      SO(4, 4, true);
    }
    *blocks_per_cu = 0;
    return hipSuccess;
  }
  if (nw == 1) {
    if (gm <= 1) SO(1, 1, false);
    if (gm <= 2) SO(2, 1, false);
    SO(4, 1, false);
  }
  if (nw == 8) {
    if (gm <= 1) SO(1, 8, false);
    if (gm <= 2) SO(2, 8, false);
    SO(4, 8, false);
  }
  if (gm <= 1) SO(1, 4, false);
  if (gm <= 2) SO(2, 4, false);
  SO(4, 4, false);
#undef SO
}
}  // namespace modal
