// 16-bit storage of a wavefield level with a per-level scale s = max |u|: stored value
// RNE(u / s) as bfloat16 or IEEE half (subnormals kept); decoded as value * s.
#pragma once

#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>

namespace awe {

__device__ __forceinline__ unsigned short enc16(float y, int bf16) {
  return bf16 ? __bfloat16_as_ushort(__float2bfloat16(y)) : __half_as_ushort(__float2half_rn(y));
}

__device__ __forceinline__ float dec16(unsigned short b, int bf16) {
  return bf16 ? __uint_as_float(((unsigned)b) << 16) : __half2float(__ushort_as_half(b));
}

// 1 / s for encoding; 0 when the level is identically zero (its codes are then 0).
__device__ __forceinline__ float inv_scale(float s) { return s > 0.f ? 1.f / s : 0.f; }

// Max over the 64 lanes of a wave (all lanes must call).
__device__ __forceinline__ float wave_max(float v) {
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

// The scale of a FULL-stored level is kept as kScaleSlots partial maxima (one per XCD,
// chosen by the workgroup id), so the per-workgroup atomic maxima of one level do not all
// serialise on one address; readers take the max of the slots.
constexpr int kScaleSlots = 8;

__device__ __forceinline__ float level_scale(const float* scl, int level) {
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < kScaleSlots; ++i) s = fmaxf(s, scl[level * kScaleSlots + i]);
  return s;
}

// One atomic max on the float bits of the N waves' maxima red (exact and order independent for
// non-negative values) into the workgroup's slot of this level; one thread calls it.
// PEEK: read the slot first and send no atomic that it already exceeds (3D).
template <int N, bool PEEK = false>
__device__ __forceinline__ void max_to_slot(const float* red, float* scl, int level) {
  float m = red[0];
  for (int w = 1; w < N; ++w) m = fmaxf(m, red[w]);
  // the atomics of a shot's level queue on one cache line, about 50 ns each: the 3600 workgroups of a
  // 240^3 step took 183 us, 69 without the store; with the peek 75.  A 2D shot has too few
  // workgroups for that, and the peek's latency showed there (1 to 3 % at 5 us a launch).  A stale
  // read only sends an atomic that changes nothing.
  unsigned* slot = reinterpret_cast<unsigned*>(scl) + level * kScaleSlots + (blockIdx.x & (kScaleSlots - 1));
  if (!PEEK || __float_as_uint(m) > __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
    atomicMax(slot, __float_as_uint(m));
}

// max_to_slot of a value per thread of a workgroup of N waves (all threads must call; uses one small LDS
// array).
template <int N, bool PEEK>
__device__ __forceinline__ void block_max_to_slot(float v, float* scl, int level) {
  __shared__ float red[N];
  v = wave_max(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) max_to_slot<N, PEEK>(red, scl, level);
}

}  // namespace awe
