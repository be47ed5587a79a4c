// Values between the lanes of a wave, and what keeps the compiler from undoing it.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace burgers {

// Whole-wave DPP move: CTRL 0x138 / 0x130 the value of lane - 1 / lane + 1 (lane 0 / lane 63 keep their own), 0x13C /
// 0x134 the same around the wave.
template <int CTRL>
__device__ __forceinline__ float wave_move(float x) {
  const int b = __builtin_bit_cast(int, x);
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(b, b, CTRL, 0xf, 0xf, false));
}
template <int CTRL>
__device__ __forceinline__ double wave_move(double x) {
  const uint64_t b = __builtin_bit_cast(uint64_t, x);
  const int lo = static_cast<int>(b & 0xffffffffu), hi = static_cast<int>(b >> 32);
  const uint32_t l = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xf, 0xf, false));
  const uint32_t h = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xf, 0xf, false));
  return __builtin_bit_cast(double, (static_cast<uint64_t>(h) << 32) | l);
}

// A binary64 value of the lane at byte address `at` (4 x lane).
__device__ __forceinline__ double lane_value(double v, int at) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(at, static_cast<int>(b & 0xffffffffu)));
  const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(at, static_cast<int>(b >> 32)));
  return __builtin_bit_cast(double, (static_cast<uint64_t>(hi) << 32) | lo);
}

// A wave's LDS accesses are performed in order; the fences keep the compiler from reordering them around an exchange
// through a region of the wave's own.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// LDS index of slot i in a region padded by one per 16.
__device__ __forceinline__ int apad(int i) { return i + (i >> 4); }

// An opaque copy of a lane value: address arithmetic built on it cannot be hoisted above this point, so per-lane
// addresses are formed in the phase that uses them rather than kept live (or spilled) across the kernel.
__device__ __forceinline__ int opaque_lane(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

}  // namespace burgers
