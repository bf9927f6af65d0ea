// The lazy update of one block of columns for one tile of 16 rows, float64 matrix cores: shared by the scalar and the
// vector-quantized column solve (not part of the C ABI).
#pragma once
#include "common.h"

namespace ptq {

// Whether pairs of column tiles share 16-byte loads: the block is a whole number of pairs, an even ldu keeps them
// aligned, and the offsets fit the buffer form.
__device__ __forceinline__ bool lazy_update_paired(int nt, int n, int64_t ldu, int mpad) {
  return (nt % 2 == 0) && (ldu % 2 == 0) && (int64_t)n * ldu * 8 < ((int64_t)1 << 31) &&
         (int64_t)n * mpad * 8 < ((int64_t)1 << 31);
}

// acc[t] = this wave's share of E[row0 .. row0 + 15, 0:i1] * U[0:i1, tile t of the block at i1]: k = 4 (kWaves it + wave)
// + lane / 16, operands of the next kDepth steps in flight while the MFMAs run.  Tile t's columns in the
// block: 16 t + lane % 16, or 32 (t / 2) + 2 (lane % 16) + t % 2 where `paired`.  i1 is a multiple of 16.
// RAGGED: the last of the nt tiles ends at column bw of the block; what lies past it repeats column bw - 1 (not `paired`).
// (lane and wave are the caller's own values: formed here once more, the loop was scheduled differently and the 4096 x 4096
// scalar solve took 1775 us against 1723.)
template <int NT, int kWaves, bool RAGGED = false>
__device__ __forceinline__ void lazy_update(const double* __restrict__ U, int64_t ldu, const double* __restrict__ errT, int mpad,
                                            int n, int i1, int nt, int row0, bool paired, int lane, int wave, f64x4 (&acc)[NT],
                                            int bw = 0) {
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
  constexpr int kDepth = (NT >= 16) ? 2 : 4;
  const int kl = lane >> 4, cl = lane & 15;
  const int wv = __builtin_amdgcn_readfirstlane(wave);   // uniform: scalar loop control
  int coff[NT];  // tiles beyond the block re-read its last tile (result unused)
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    coff[t] = 16 * (t < nt ? t : nt - 1);
    if constexpr (RAGGED) coff[t] = min(coff[t] + cl, bw - 1) - cl;
  }
  const int niter = (i1 - 4 * wv + 4 * kWaves - 1) / (4 * kWaves);  // k = 32 it + 4 wave + kl < i1 (a multiple of 16)
  double av[kDepth], bv[kDepth][NT];
  auto mfmas = [&](int d) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
      acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[d], bv[d][t], acc[t], 0, 0, 0);
  };
  // The loop: slot d's MFMAs, then the request for the step kDepth later into the same slot.  In the
  // steady state there is no branch between the first request and the last iteration, every slot is
  // valid and has a successor, and the requests are buffer loads whose per-lane offsets never change
  // (the step advances in a scalar offset: no address arithmetic between the MFMAs).
  auto run = [&](auto issue) {
    int it = 0;
    if (niter >= 2 * kDepth) {
#pragma unroll
      for (int d = 0; d < kDepth; ++d) issue(d, d);
      for (; it + 2 * kDepth <= niter; it += kDepth) {
#pragma unroll
        for (int d = 0; d < kDepth; ++d) {
          mfmas(d);
          issue(d, it + d + kDepth);
        }
      }
    } else {
#pragma unroll
      for (int d = 0; d < kDepth; ++d)
        if (d < niter) issue(d, d);
    }
    for (; it < niter; it += kDepth) {
#pragma unroll
      for (int d = 0; d < kDepth; ++d) {
        if (it + d < niter) {
          mfmas(d);
          if (it + d + kDepth < niter) issue(d, it + d + kDepth);
        }
      }
    }
  };
  const bool offsets32 = (int64_t)n * ldu * 8 < ((int64_t)1 << 31) && (int64_t)n * mpad * 8 < ((int64_t)1 << 31);
  if (offsets32) {
    const __amdgpu_buffer_rsrc_t re = __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(errT + row0), 0,
                                                                        (int)0xFFFFFFFFu, 0x00020000);
    const __amdgpu_buffer_rsrc_t ru = __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(U + i1), 0,
                                                                        (int)0xFFFFFFFFu, 0x00020000);
    const int ve = ((4 * wv + kl) * mpad + cl) * 8;
    const int se = 4 * kWaves * mpad * 8, su = 4 * kWaves * (int)ldu * 8;
    if (paired) {
      // The address unit takes a wave's load in 16 steps of four lanes whatever the width, so 8-byte
      // loads top out at 32 bytes per clock and compute unit -- less than the eight MFMAs of a k-step
      // need.  A lane therefore fetches two neighbouring columns at once (16 bytes) and gives one to each
      // of a pair of tiles: tile 2p + q works on columns 32 p + 2 cl + q.  The MFMA does not care which
      // columns make up a tile; the partial sums go back to their columns through the same map.
      int vu[NT / 2];
#pragma unroll
      for (int p = 0; p < NT / 2; ++p) vu[p] = ((4 * wv + kl) * (int)ldu + 2 * cl + (coff[2 * p] & ~31)) * 8;
      typedef double f64x2 __attribute__((ext_vector_type(2)));
      run([&](int slot, int it) {
        av[slot] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(re, ve, it * se, 0));
#pragma unroll
        for (int p = 0; p < NT / 2; ++p) {
          const f64x2 two = __builtin_bit_cast(f64x2, __builtin_amdgcn_raw_buffer_load_b128(ru, vu[p], it * su, 0));
          bv[slot][2 * p] = two[0];
          bv[slot][2 * p + 1] = two[1];
        }
      });
    } else {
      int vu[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) vu[t] = ((4 * wv + kl) * (int)ldu + cl + coff[t]) * 8;
      run([&](int slot, int it) {
        av[slot] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(re, ve, it * se, 0));
#pragma unroll
        for (int t = 0; t < NT; ++t)
          bv[slot][t] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(ru, vu[t], it * su, 0));
      });
    }
  } else {
    const double* ep = errT + (int64_t)(4 * wv + kl) * mpad + row0 + cl;
    const double* up = U + (int64_t)(4 * wv + kl) * ldu + i1 + cl;
    run([&](int slot, int it) {
      av[slot] = ep[(int64_t)it * (4 * kWaves) * mpad];
      const double* u = up + (int64_t)it * (4 * kWaves) * ldu;
#pragma unroll
      for (int t = 0; t < NT; ++t) bv[slot][t] = u[coff[t]];
    });
  }
}

}  // namespace ptq
