// The Walsh-Hadamard transform of a 256-element chunk held by one wave (not part of the C ABI): shared by the rotation
// of weights and Hessians (lopro.hip) and of the activations that enter a stored layer (artifact.hip).
#pragma once
#include "common.h"

namespace ptq {

__device__ __forceinline__ int ilog2(int x) { return 31 - __clz(x); }

// first = {a of the lower, b of the lower}, second = {a of the upper, b of the upper} half of each pair of rows of 16
// lanes (HALF: of the two halves of 32): the lower lanes of a pair hold a's two values, the upper ones b's
template <bool HALF>
__device__ __forceinline__ void lane_pair(double a, double b, double& first, double& second) {
  const unsigned long long ab = __double_as_longlong(a), bb = __double_as_longlong(b);
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  u32x2 l, h;
  if constexpr (HALF) {
    l = __builtin_amdgcn_permlane32_swap((unsigned)ab, (unsigned)bb, false, false);
    h = __builtin_amdgcn_permlane32_swap((unsigned)(ab >> 32), (unsigned)(bb >> 32), false, false);
  } else {
    l = __builtin_amdgcn_permlane16_swap((unsigned)ab, (unsigned)bb, false, false);
    h = __builtin_amdgcn_permlane16_swap((unsigned)(ab >> 32), (unsigned)(bb >> 32), false, false);
  }
  first = __longlong_as_double((long long)(((unsigned long long)h[0] << 32) | l[0]));
  second = __longlong_as_double((long long)(((unsigned long long)h[1] << 32) | l[1]));
}

constexpr int kDppReverseQuad = 0x1B;   // quad_perm [3, 2, 1, 0]: lane ^ 3
constexpr int kDppRotate8 = 0x128;      // row_ror:8: lane ^ 8

// Walsh-Hadamard transform (natural order, unscaled) of blocks of 2^lg consecutive elements of a 256-element
// chunk held four per lane, element 4 * lane + i in v[i]; 2 <= lg <= 8.  Two stages in registers, six across lanes by
// data-parallel primitives and row swaps (no trip through the LDS crossbar): lane l gets v + partner where its bit of
// the stage is clear, partner - v where it is set.
__device__ __forceinline__ void fwht_chunk(double (&v)[4], int lg, int lane) {
  {
    const double a = v[0] + v[1], b = v[0] - v[1], c = v[2] + v[3], d = v[2] - v[3];
    v[0] = a + c;
    v[1] = b + d;
    v[2] = a - c;
    v[3] = b - d;
  }
  if (lg > 2) {
    const double sign = lane & 1 ? -1.0 : 1.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = fma(sign, v[i], dpp_move<kDppSwapPairs>(v[i]));
  }
  if (lg > 3) {
    const double sign = lane & 2 ? -1.0 : 1.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = fma(sign, v[i], dpp_move<kDppSwapHalfQuads>(v[i]));
  }
  if (lg > 4) {   // lane ^ 4 = (lane ^ 7) ^ 3
    const double sign = lane & 4 ? -1.0 : 1.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = fma(sign, v[i], dpp_move<kDppReverseQuad>(dpp_move<kDppHalfMirror>(v[i])));
  }
  if (lg > 5) {
    const double sign = lane & 8 ? -1.0 : 1.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = fma(sign, v[i], dpp_move<kDppRotate8>(v[i]));
  }
  if (lg > 6) {
    const double sign = lane & 16 ? -1.0 : 1.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      double a, b;
      lane_pair<false>(v[i], v[i], a, b);
      v[i] = fma(sign, b, a);
    }
  }
  if (lg > 7) {
    const double sign = lane & 32 ? -1.0 : 1.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      double a, b;
      lane_pair<true>(v[i], v[i], a, b);
      v[i] = fma(sign, b, a);
    }
  }
}

}  // namespace ptq
