// Merge of a row's key-range splits: the arithmetic shared by the merge kernel
// and the short-sequence kernel, so that both give the same bits.
#pragma once

#include "fwd_kernel.hpp"

namespace attn {

template <int DT>
__device__ __forceinline__ float widen(uint16_t h) {
  if constexpr (DT == ATTN_BF16) return __builtin_bit_cast(float, (uint32_t)h << 16);
  else return (float)__builtin_bit_cast(_Float16, h);
}

// Eight output columns of one row from its n splits' references and sums
// (st) and normalised partial outputs (po).  NS >= n is a compile-time bound;
// the slots past n repeat slot n - 1 and take weight 0, which leaves the
// maximum, the sum and the accumulator unchanged.
template <int DT, int NS>
__device__ __forceinline__ u32x4_t merge_splits(const float2 (&st)[NS], const u32x4_t (&po)[NS], int n) {
  using S = typename Mfma<DT>::S;
  float m = -INFINITY;
#pragma unroll
  for (int s = 0; s < NS; ++s) m = fmaxf(m, st[s].x);
  float lt = 0.f;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const float wgt = (s >= n || st[s].x == -INFINITY) ? 0.f : st[s].y * exp2_hw(st[s].x - m);
    lt += wgt;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      acc[2 * e] += wgt * widen<DT>((uint16_t)(po[s][e] & 0xffffu));
      acc[2 * e + 1] += wgt * widen<DT>((uint16_t)(po[s][e] >> 16));
    }
  }
  const float inv = lt > 0.f ? 1.f / lt : 0.f;
  uint32_t out[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const S a = (S)(acc[2 * e] * inv), b = (S)(acc[2 * e + 1] * inv);
    out[e] = (uint32_t)__builtin_bit_cast(uint16_t, a) | ((uint32_t)__builtin_bit_cast(uint16_t, b) << 16);
  }
  return (u32x4_t){out[0], out[1], out[2], out[3]};
}

}  // namespace attn
