// Sums over the 64 lanes of a wave in a fixed order.
#pragma once

#include "common.h"

namespace chefsi {

// v[i] summed over the 64 lanes for every i < N (N a power of two, at most 64): each of the
// first log2 N exchanges halves the values a lane keeps, so lane l ends with the sum of
// value l / (64 / N) in v[0] after N - 1 + log2(64 / N) exchanges (6 N for N plain sums).
template <int M, int OFF, typename T, int N>
__device__ __forceinline__ void wave_sums_step(T (&v)[N], int lane) {
  if constexpr (M >= 1) {
    const bool up = lane & OFF;
#pragma unroll
    for (int i = 0; i < M; ++i) {
      const T keep = up ? v[i + M] : v[i];
      const T give = up ? v[i] : v[i + M];
      v[i] = keep + __shfl_xor(give, OFF, 64);
    }
    wave_sums_step<M / 2, OFF / 2>(v, lane);
  } else if constexpr (OFF >= 1) {
    v[0] += __shfl_xor(v[0], OFF, 64);
    wave_sums_step<0, OFF / 2>(v, lane);
  }
}
template <typename T, int N>
__device__ __forceinline__ void wave_sums(T (&v)[N], int lane) {
  wave_sums_step<N / 2, 32>(v, lane);
}

}  // namespace chefsi
