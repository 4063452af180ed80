// Device helpers shared by the forward and reverse kernels (gfx950).
#pragma once
#include <hip/hip_runtime.h>

#include "kernels.h"

namespace modal {

// The absolute index of a launch's first step: given by the host, in which
// case one thread stores the next launch's (step_done), or read from the
// device's counter, which another launch then advances (captured launches,
// whose replays the host does not see).
template <class P>
__device__ __forceinline__ long long step_first(const P& p) {
  return p.base >= 0 ? p.base : *p.step_base;
}
template <class P>
__device__ __forceinline__ void step_done(const P& p) {
  if (p.base >= 0 && blockIdx.x == 0 && threadIdx.x == 0) *p.step_base = p.base + p.n_steps;
}

// d+ = m X - p d + r fe ;  X+ = X + d+, in FP64: four instructions at the
// FP32 issue rate (gfx950 runs FP64 vector code at the rate of unpacked
// FP32), where the float-float form of this update took about 80 and filled
// most of a small instance's step (one-wave string: 0.30 us a step before).
__device__ __forceinline__ void mode_step(double& x, double& d, double m, double p, double r, float fe) {
  d = fma(m, x, fma(-p, d, r * (double)fe));
  x += d;
}

// ------------------------------------------------------------------ helpers
// Data-parallel move between lanes of a 16-lane row (DPP control word C).
template <int C>
__device__ __forceinline__ float dpp_mov(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), C, 0xF, 0xF, true));
}
__device__ __forceinline__ float lane_value(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
// Sum over the 64 lanes of a wave (all lanes active), the same on every lane.
// Within each 16-lane row four DPP exchanges (partner lane ^1, ^2, the mirror
// within 8 lanes, the mirror within 16) leave the row's sum on all its lanes,
// identical bits on each since every pairing is symmetric; the four row sums
// are then read out and added.  No LDS crossbar round trips, unlike a
// shuffle-based butterfly.
__device__ __forceinline__ float wave_sum(float v) {
  v += dpp_mov<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp_mov<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp_mov<0x141>(v);  // row_half_mirror
  v += dpp_mov<0x140>(v);  // row_mirror
  return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}
// Sums of v over each group of L consecutive lanes (L = 16, 32 or 64), the
// same bits on every lane of a group: the DPP exchanges of wave_sum within a
// row, then gfx950's lane swaps between rows and halves.
template <int L>
__device__ __forceinline__ float group_sum(float v) {
  v += dpp_mov<0xB1>(v);
  v += dpp_mov<0x4E>(v);
  v += dpp_mov<0x141>(v);
  v += dpp_mov<0x140>(v);
  if constexpr (L >= 32) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  if constexpr (L >= 64) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  return v;
}
// c . x of each quad of lanes, on its last lane (zero on the others), rounded
// as dot4 rounds four elements of one lane
__device__ __forceinline__ float quad_dot(float c, float x, int lane) {
  float v = c * x;
#pragma unroll
  for (int j = 1; j < 4; ++j) {
    const float t = fmaf(c, x, dpp_mov<0x90>(v));  // quad_perm [0,0,1,2]: the lane before
    v = (lane & 3) == j ? t : v;
  }
  return (lane & 3) == 3 ? v : 0.f;
}
// Sum of N values (a power of two) as a tree.
template <int N>
__device__ __forceinline__ float tree_sum(float (&v)[N]) {
#pragma unroll
  for (int s = N / 2; s > 0; s /= 2)
#pragma unroll
    for (int w = 0; w < s; ++w) v[w] += v[w + s];
  return v[0];
}
// Sum of v over the four lanes l, l^16, l^32, l^48 (gfx950 lane swaps).
__device__ __forceinline__ float quad_sum(float v) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  auto q = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(q[0]) + __uint_as_float(q[1]);
}
// Lane j of each group of L lanes (j the same for every group).
template <int L>
__device__ __forceinline__ float group_lane(float v, int j) {
  if constexpr (L == 64) return lane_value(v, j);
  return __shfl(v, j, L);
}
__device__ __forceinline__ float4 f4(float v) { return make_float4(v, v, v, v); }
__device__ __forceinline__ float4 fma4(float4 a, float b, float4 c) {
  return make_float4(fmaf(a.x, b, c.x), fmaf(a.y, b, c.y), fmaf(a.z, b, c.z), fmaf(a.w, b, c.w));
}
__device__ __forceinline__ float4 add4(float4 a, float4 b) {
  return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
}
__device__ __forceinline__ float dot4(float4 a, float4 b) {
  return fmaf(a.w, b.w, fmaf(a.z, b.z, fmaf(a.y, b.y, a.x * b.x)));
}
__device__ __forceinline__ float4 ld4(const float* p) { return *reinterpret_cast<const float4*>(p); }

typedef double v2d __attribute__((ext_vector_type(2)));
// four consecutive doubles (two 16-byte accesses; p on a multiple of 16 bytes)
struct f64x4 {
  double v[4];
};
__device__ __forceinline__ f64x4 ld4d(const double* p) {
  const v2d a = reinterpret_cast<const v2d*>(p)[0], b = reinterpret_cast<const v2d*>(p)[1];
  return {{a.x, a.y, b.x, b.y}};
}
__device__ __forceinline__ void st4d(double* p, const f64x4& v) {
  reinterpret_cast<v2d*>(p)[0] = (v2d){v.v[0], v.v[1]};
  reinterpret_cast<v2d*>(p)[1] = (v2d){v.v[2], v.v[3]};
}
// their FP32 roundings
__device__ __forceinline__ float4 to_f4(const f64x4& v) {
  return make_float4((float)v.v[0], (float)v.v[1], (float)v.v[2], (float)v.v[3]);
}

typedef float v4f __attribute__((ext_vector_type(4)));
// Raw buffer resource over `bytes` bytes at p (stride 0).  Loads at byte
// offsets >= bytes are out of range and return zeros without a memory
// access; the last word is the standard gfx9 raw-buffer format word.  The
// callers' values are wave-uniform; readfirstlane states it so that the
// resource lives in scalar registers.
typedef int v4i __attribute__((ext_vector_type(4)));
__device__ __forceinline__ v4i buf_rsrc(const float* p, int bytes) {
  const unsigned long long a = reinterpret_cast<unsigned long long>(p);
  v4i r;
  r.x = __builtin_amdgcn_readfirstlane((int)(unsigned)a);
  r.y = __builtin_amdgcn_readfirstlane((int)((a >> 32) & 0xffffu));
  r.z = __builtin_amdgcn_readfirstlane(bytes);
  r.w = 0x00020000;
  return r;
}
// The LLVM raw buffer load intrinsic, declared directly.
__device__ v4f llvm_raw_buffer_load_v4f32(v4i rsrc, int voffset, int soffset, int aux)
    __asm("llvm.amdgcn.raw.buffer.load.v4f32");
// The partial forces that the slabs of a split instance exchange in global
// memory are written and read with the sc1 cache policy, which gfx950 keeps
// coherent across the XCDs' separate L2 caches: the policy of an agent-scope
// relaxed atomic access, here on 16-byte buffer accesses instead of four
// separate 4-byte atomics.  Publishing a partial then needs only a wait for
// its stores to complete before the arrival word (an agent-scope atomic) is
// stored, and reading one needs no L2 invalidation: an agent-scope release or
// acquire fence would write back or invalidate the whole L2 of the XCD on
// every step.  The resource spans one instance's exchange region (offsets
// past it read zeros and drop stores); byte offsets per lane.
constexpr int kCoherentPolicy = 16;  // sc1 bit of the buffer instructions' cache-policy operand
__device__ void llvm_raw_buffer_store_v4f32(v4f v, v4i rsrc, int voffset, int soffset, int aux)
    __asm("llvm.amdgcn.raw.buffer.store.v4f32");
__device__ __forceinline__ void st4_coherent(v4i r, int byte_off, float4 v) {
  v4f w;
  w.x = v.x;
  w.y = v.y;
  w.z = v.z;
  w.w = v.w;
  llvm_raw_buffer_store_v4f32(w, r, byte_off, 0, kCoherentPolicy);
}
__device__ __forceinline__ float4 ld4_coherent(v4i r, int byte_off) {
  const v4f v = llvm_raw_buffer_load_v4f32(r, byte_off, 0, kCoherentPolicy);
  return make_float4(v.x, v.y, v.z, v.w);
}
// After a wave's partial-force stores (st4_coherent): waits until the memory
// system has acknowledged them, so that an arrival word stored afterwards
// cannot be seen before them.  A workgroup-scope release fence emits no such
// wait when a workgroup's waves share one CU, and an agent-scope one would
// also write back the XCD's whole L2; the wait on the vector-memory counter
// alone is what the exchange needs.  It is also a compiler barrier, and waits
// for loads as well.
__device__ __forceinline__ void publish_fence() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
// Before reading partials (ld4_coherent) once the words have been seen:
// keeps the compiler from moving the reads above the words' loads (the
// hardware issues them after the polling loop, whose exit depends on the
// words' values).
__device__ __forceinline__ void consume_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup"); }

// sum over t = t0, t0 + dt, ... (t < n) of the float4 at byte offset
// off + t * stride of resource r (partial forces of other workgroups, read
// coherently), eight reads issued before the first add (sixteen measured
// slower); a fixed order, so every caller gets the same bits
__device__ __forceinline__ float4 sum_slabs4_coherent(v4i r, int off, int t0, int dt, int n, int stride) {
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  int t = t0;
  for (; t + 7 * dt < n; t += 8 * dt) {
    float4 a[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) a[i] = ld4_coherent(r, off + (t + i * dt) * stride);
#pragma unroll
    for (int i = 0; i < 8; ++i) s = add4(s, a[i]);
  }
  for (; t < n; t += dt) s = add4(s, ld4_coherent(r, off + t * stride));
  return s;
}

// sum over t < n of the float4 at p + t * stride (LDS), with four partial
// sums so that four reads are in flight before the first add waits
__device__ __forceinline__ float4 sum_strided4(const float* p, int n, int stride) {
  float4 s0 = ld4(p), s1 = make_float4(0.f, 0.f, 0.f, 0.f), s2 = s1, s3 = s1;
  int t = 1;
  for (; t + 3 < n; t += 4) {
    s1 = add4(s1, ld4(p + t * stride));
    s2 = add4(s2, ld4(p + (t + 1) * stride));
    s3 = add4(s3, ld4(p + (t + 2) * stride));
    s0 = add4(s0, ld4(p + (t + 3) * stride));
  }
  for (; t < n; ++t) s1 = add4(s1, ld4(p + t * stride));
  return add4(add4(s0, s1), add4(s2, s3));
}

// sum of n consecutive floats (LDS), four partial sums
__device__ __forceinline__ float sum_run(const float* p, int n) {
  float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
  int c = 0;
  for (; c + 3 < n; c += 4) {
    s0 += p[c];
    s1 += p[c + 1];
    s2 += p[c + 2];
    s3 += p[c + 3];
  }
  for (; c < n; ++c) s0 += p[c];
  return (s0 + s1) + (s2 + s3);
}
__device__ __forceinline__ void st4(float* p, float4 v) { *reinterpret_cast<float4*>(p) = v; }

// 16-byte load through a buffer resource with cache policy POL: kStream,
// the non-temporal hint, for tensors streamed from HBM once per step (the
// batch), or kKeep, the default policy, for a latency-bound instance whose
// tensor stays in the caches from step to step (measured on a lone 200/200
// plate: forward 14.0 -> 12.1 us and reverse 18.2 -> 16.8 us per step; the
// 256-plate batch 233 -> 247 ms per launch with kKeep).
constexpr int kStream = 2, kKeep = 0;
template <int POL = kStream>
__device__ __forceinline__ float4 buf_ld4(v4i r, int voff) {
  const v4f v = llvm_raw_buffer_load_v4f32(r, voff, 0, POL);
  return make_float4(v.x, v.y, v.z, v.w);
}

// 4-byte load through a buffer resource (zero at out-of-range offsets)
__device__ float llvm_raw_buffer_load_f32(v4i rsrc, int voffset, int soffset, int aux)
    __asm("llvm.amdgcn.raw.buffer.load.f32");
__device__ __forceinline__ float buf_ld1(v4i r, int voff) { return llvm_raw_buffer_load_f32(r, voff, 0, 0); }

// Orders this wave's LDS writes before its later LDS reads by other lanes.
// Workgroups are single waves, so no s_barrier is needed, and vector-memory
// loads in flight are not waited for.
__device__ __forceinline__ void wave_lds_sync() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_wave_barrier();
}

// Workgroup barrier for LDS traffic only: this wave's LDS operations are
// complete and every wave has arrived.  Unlike __syncthreads it does not
// wait for outstanding global loads, so prefetches stay in flight across it.
__device__ __forceinline__ void block_lds_sync() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}


// Waits until every slab's arrival word f[t] (t < nslab) has reached
// `target` (wrap-safe); called by a whole wave, whose lanes poll the words
// together, so that no slab's arrival waits on another's (each slab stores
// its own word; nothing is read-modify-written).  Returns false if the wait
// was abandoned (after `timeout` ticks here, or elsewhere).
__device__ inline bool wait_slabs(const unsigned int* f, int nslab, unsigned int target, int* flags,
                                  unsigned long long timeout) {
  const int lane = threadIdx.x & (kWave - 1);
  const unsigned long long t0 = wall_clock64();
  while (true) {
    bool ok = true;
    for (int t = lane; t < nslab; t += kWave) {
      const unsigned int v = __hip_atomic_load(f + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      ok = ok && (int)(v - target) >= 0;
    }
    if (__all(ok)) return true;
    if (__hip_atomic_load(&flags[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return false;
    if (wall_clock64() - t0 > timeout) {
      __hip_atomic_store(&flags[0], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return false;
    }
    __builtin_amdgcn_s_sleep(2);
  }
}

}  // namespace modal
