// Shared by the on-chip kernels (chip_kernel.hip, chip_grad_kernel.hip): the
// register tiles, the row sums and the shapes that have a kernel.
#pragma once
#include <hip/hip_runtime.h>

#include "device_common.h"
#include "kernels.h"

namespace modal {

// Row index whose sum row_sums leaves on lane l: l & (rows rounded up to a
// power of two, at least 4, - 1).
__host__ __device__ constexpr int row_lanes(int r) { return r <= 4 ? 4 : (r <= 8 ? 8 : 16); }

// Lane l - N of its 16-lane row (rotation).
template <int N>
__device__ __forceinline__ float row_ror(float v) {
  return dpp_mov<0x120 + N>(v);
}

// R sums over the 64 lanes (R <= 16), transposed: lane l gets the sum of
// v[l & (row_lanes(R) - 1)].  Four rows join into one value in two exchanges
// within quads (lane bits 0 and 1 choose the row), up to four such values in
// two rotations of the 16-lane row (bits 2 and 3), and one value crosses the
// rows and halves: 17, 28 or 48 instructions for 4, 8 or 16 rows, where a
// full sum of each row takes 11.
template <int R>
__device__ __forceinline__ float row_sums(const float (&v)[R], int lane) {
  constexpr int NQ = row_lanes(R) / 4;
  const bool b0 = lane & 1, b1 = lane & 2, b2 = lane & 4, b3 = lane & 8;
  float q[NQ];
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    float a[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) a[j] = 4 * i + j < R ? v[4 * i + j] : 0.f;
    const float e = (b0 ? a[1] : a[0]) + dpp_mov<0xB1>(b0 ? a[0] : a[1]);
    const float o = (b0 ? a[3] : a[2]) + dpp_mov<0xB1>(b0 ? a[2] : a[3]);
    q[i] = (b1 ? o : e) + dpp_mov<0x4E>(b1 ? e : o);
  }
  float t;
  if constexpr (NQ == 1) {
    t = q[0] + row_ror<4>(q[0]);
    t += row_ror<8>(t);
  } else if constexpr (NQ == 2) {
    t = (b2 ? q[1] : q[0]) + row_ror<4>(b2 ? q[0] : q[1]);
    t += row_ror<8>(t);
  } else {
    const float e = (b2 ? q[1] : q[0]) + row_ror<4>(b2 ? q[0] : q[1]);
    const float o = (b2 ? q[3] : q[2]) + row_ror<4>(b2 ? q[2] : q[3]);
    t = (b3 ? o : e) + row_ror<8>(b3 ? e : o);
  }
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(t), __float_as_uint(t), false, false);
  t = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(t), __float_as_uint(t), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Loads one wave's tensor tile: put(r, t, value) gets, for every row r < R and
// column t < W, Ht[row r][perm[jb + t]][lane's mode], t < jl, zero elsewhere
// (through a buffer resource over the instance's tensor, whose out-of-range
// offsets read zeros: no branches).
template <int W, int R, class Put>
__device__ __forceinline__ void chip_load(const ChipMap& M, const InstDev& I, const float* H, int wave, int k, int jb,
                                          int jl, Put put) {
  const long long row = (long long)I.nt * I.ntp;
  const bool vk = I.kind == KIND_VK;
  const v4i rs = buf_rsrc(H + I.h_off, vk ? (int)(4 * I.nin * row) : 0);
#pragma unroll
  for (int t = 0; t < W; ++t) {
    const int j = M.perm[min(jb + t, kWave - 1)];
    const bool live = vk && k >= 0 && t < jl && j >= 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int n = M.row[wave][r];
      put(r, t, buf_ld1(rs, live && n >= 0 ? 4 * (int)(n * row + j * I.ntp + k) : 0x7fffffff));
    }
  }
}

// acc[r] += sum_t h[r][t] x[t], x in LDS on a multiple of 16 bytes
template <int W, int R>
__device__ __forceinline__ void chip_mul(float (&acc)[R], const float (&h)[R][W], const float* x) {
#pragma unroll
  for (int t4 = 0; t4 < W / 4; ++t4) {
    const float4 q = ld4(x + 4 * t4);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      acc[r] = fmaf(h[r][4 * t4], q.x, acc[r]);
      acc[r] = fmaf(h[r][4 * t4 + 1], q.y, acc[r]);
      acc[r] = fmaf(h[r][4 * t4 + 2], q.z, acc[r]);
      acc[r] = fmaf(h[r][4 * t4 + 3], q.w, acc[r]);
    }
  }
}

// The same against two vectors, x and u, for tiles that leave few registers:
// one column group at a time, the next group's reads of x and u issued before
// its products; columns [0, WR) from the registers h, [WR, W) from LDS, where
// hl holds this lane's float4 of each (group, row).
template <int W, int WR, int R>
__device__ __forceinline__ void chip_mul2(float (&V)[R], float (&Wv)[R], const float (&h)[R][WR], const float* hl,
                                          const float* x, const float* u) {
  float4 xc = ld4(x), uc = ld4(u);
#pragma unroll
  for (int t4 = 0; t4 < W / 4; ++t4) {
    float4 xn = xc, un = uc;
    if (t4 + 1 < W / 4) {
      xn = ld4(x + 4 * t4 + 4);
      un = ld4(u + 4 * t4 + 4);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      float4 hv;
      if (4 * t4 < WR) hv = make_float4(h[r][4 * t4 % WR], h[r][(4 * t4 + 1) % WR], h[r][(4 * t4 + 2) % WR], h[r][(4 * t4 + 3) % WR]);
      else hv = ld4(hl + ((t4 - WR / 4) * R + r) * 4 * kWave);
      V[r] = fmaf(hv.w, xc.w, fmaf(hv.z, xc.z, fmaf(hv.y, xc.y, fmaf(hv.x, xc.x, V[r]))));
      Wv[r] = fmaf(hv.w, uc.w, fmaf(hv.z, uc.z, fmaf(hv.y, uc.y, fmaf(hv.x, uc.x, Wv[r]))));
    }
    xc = xn;
    uc = un;
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Sum over the waves of red[w][lane], in a fixed order, so that every wave
// gets the same bits.
__device__ __forceinline__ float wave_join(const float (*red)[kWave], int lane) {
  float v[kChipWaves];
#pragma unroll
  for (int w = 0; w < kChipWaves; ++w) v[w] = red[w][lane];
  return tree_sum(v);
}

// Lane stride of a vector of modes in LDS: a run of W <= 64 columns from any
// lane stays inside it, and reads zeros past the modes.
constexpr int kChipVec = 2 * kWave;

// Columns and rows per wave that have a kernel (W R <= kChipTile floats per
// lane: with the rest of the kernel's registers 256 and two waves per SIMD; the
// forward kernel that records spills 12, 44 and 20 bytes a lane at 16 x 12,
// 20 x 10 and 40 x 5).
constexpr int kChipTile = 200;
#define CHIP_SHAPES(X)                                                                            \
  X(8, 1) X(8, 2) X(8, 3) X(8, 4) X(8, 5) X(8, 6) X(8, 7) X(8, 8) X(8, 10) X(8, 12)               \
  X(12, 1) X(12, 2) X(12, 3) X(12, 4) X(12, 5) X(12, 6) X(12, 7) X(12, 8) X(12, 10) X(12, 12)     \
  X(16, 1) X(16, 2) X(16, 3) X(16, 4) X(16, 5) X(16, 6) X(16, 7) X(16, 8) X(16, 10) X(16, 12)     \
  X(20, 1) X(20, 2) X(20, 3) X(20, 4) X(20, 5) X(20, 6) X(20, 7) X(20, 8) X(20, 10)               \
  X(24, 1) X(24, 2) X(24, 3) X(24, 4) X(24, 5) X(24, 6) X(24, 7) X(24, 8)                         \
  X(32, 1) X(32, 2) X(32, 3) X(32, 4) X(32, 5) X(32, 6)                                           \
  X(40, 1) X(40, 2) X(40, 3) X(40, 4) X(40, 5)                                                    \
  X(48, 1) X(48, 2) X(48, 3) X(48, 4)                                                             \
  X(64, 1) X(64, 2) X(64, 3)

}  // namespace modal
