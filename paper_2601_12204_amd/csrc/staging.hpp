// Rows of a system passed between HBM and LDS in coalesced order.
#pragma once

#include <hip/hip_runtime.h>

#include "internal.hpp"
#include "wave.hpp"

namespace burgers {

constexpr int kRedChunk = 16;     // chunk length in the partition levels

// Rows staged in LDS are padded by one element every 32 rows: a thread reads its chunk with a lane
// stride of q rows, and without the pad q = 16 or 32 would put every lane of a wave on one bank.
__device__ __forceinline__ int padded(int i) { return i + (i >> 5); }
constexpr int padded_size(int rows) { return rows + rows / 32 + 1; }

// Coalesced copies of a block's rows between HBM and LDS: all loads are issued before the first LDS
// store, so a wave has its whole share of the block in flight at once.
template <typename S, int NT = kReduceBlock, int J = kRedChunk>
__device__ __forceinline__ void stage_in(S* stage, const S* __restrict__ src, int cnt) {
  S v[J];
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int i = static_cast<int>(threadIdx.x) + j * NT;
    v[j] = i < cnt ? src[i] : S(0);
  }
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int i = static_cast<int>(threadIdx.x) + j * NT;
    if (i < cnt) stage[padded(i)] = v[j];
  }
}

template <typename S, int NT = kReduceBlock, int J = kRedChunk>
__device__ __forceinline__ void stage_out(const S* stage, S* __restrict__ dst, int cnt) {
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int i = static_cast<int>(threadIdx.x) + j * NT;
    if (i < cnt) dst[i] = stage[padded(i)];
  }
}

// Crank-Nicolson store: the staged rows hold the half-dt BTCS solution y; write 2 y - u, with u re-read
// (coalesced) from the old state.
template <typename S, int NT = kReduceBlock, int J = kRedChunk>
__device__ __forceinline__ void stage_out_cn(const S* stage, const S* __restrict__ old, S* __restrict__ dst,
                                             int cnt) {
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int i = static_cast<int>(threadIdx.x) + j * NT;
    if (i < cnt)
      dst[i] = static_cast<S>(2.0 * static_cast<double>(stage[padded(i)]) - static_cast<double>(old[i]));
  }
}

}  // namespace burgers
