// What is stored for a layer and the form it is applied in (paper Sec. 3.2, Eq. 7; Sec. 3.4,
// Eq. 12; Algorithm 1, last lines; the time-complexity appendix):
//   * bit packing of the codes and its inverse with dequantization;
//   * the layer applied to a few tokens:  O = X~ Dequant(W_q)^T + ((X diag(s)^-1) V^T diag(sigma)) U,
//     X~ = X P Q  (the input is permuted and rotated once, the residual is never rotated back).
//
// Packing: 32 consecutive codes of a row (a chunk) form a little-endian bit stream of exactly d
// 32-bit words, code j in bits [j d, (j+1) d); the chunks are stored chunk-major,
// packed[chunk][row][d], and the grids group-major, scale[group][row] and zero[group][row], so
// that lanes that work on consecutive rows read consecutive memory.
//
// The product with the packed residual takes two forms: a few tokens row by row on the vector unit (bound by the
// codes' stream from memory), more of them in tiles on the 16-bit matrix cores.
#include <limits.h>

#include <algorithm>
#include <cmath>

#include "common.h"
#include "lds_dma.h"
#include "rotation.h"

namespace ptq {
namespace {

constexpr int kChunk = 32;   // codes per lane and step: d words

// Code j of a chunk from its d words; j and d are compile-time constants, so this is one
// bit-field extract, or two shifts and a mask where a 3-bit code straddles two words.
template <int BITS>
__device__ __forceinline__ uint32_t chunk_code(const uint32_t* __restrict__ words, int j) {
  const int pos = j * BITS, wi = pos >> 5, sh = pos & 31;
  constexpr uint32_t mask = (1u << BITS) - 1u;
  if (sh + BITS <= 32) return (words[wi] >> sh) & mask;
  return ((words[wi] >> sh) | (words[wi + 1] << (32 - sh))) & mask;
}

template <int BITS>
__device__ __forceinline__ void unpack_chunk(const uint32_t* __restrict__ words, uint8_t (&code)[kChunk]) {
#pragma unroll
  for (int j = 0; j < kChunk; ++j) code[j] = (uint8_t)chunk_code<BITS>(words, j);
}

// scale[row][group] -> scale[group][row], the same for the zero-points: 32 x 32 tiles through LDS
struct GridTranspose {
  const float* scales;
  const uint8_t* zeros;
  int ng;
  float* scales_t;
  uint8_t* zeros_t;
  int row_tiles, tiles;   // tiles = 0: nothing to do
};

__device__ __forceinline__ void transpose_grids_tile(const GridTranspose& a, int m, int tile) {
  __shared__ float ts[32][33];
  __shared__ uint8_t tz[32][33];
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const int r0 = (tile % a.row_tiles) * 32, g0 = (tile / a.row_tiles) * 32;
  for (int k = ty; k < 32; k += 8) {
    const int row = r0 + k, g = g0 + tx;
    if (row < m && g < a.ng) { ts[k][tx] = a.scales[(int64_t)row * a.ng + g]; tz[k][tx] = a.zeros[(int64_t)row * a.ng + g]; }
  }
  __syncthreads();
  for (int k = ty; k < 32; k += 8) {
    const int g = g0 + k, row = r0 + tx;
    if (row < m && g < a.ng) { a.scales_t[(int64_t)g * m + row] = ts[tx][k]; a.zeros_t[(int64_t)g * m + row] = tz[tx][k]; }
  }
}

// The last grids.tiles workgroups bring the grids into their order (one launch instead of two: a call of 512 x 512 codes
// 11.3 -> 6.6 us, of 11008 x 4096 31.3 -> 29.5).
template <int BITS>
__global__ __launch_bounds__(256) void pack_kernel(const uint8_t* __restrict__ codes, int64_t ldc, int m, int n,
                                                   uint32_t* __restrict__ packed, GridTranspose grids) {
  const int pack_blocks = (int)gridDim.x - grids.tiles;
  if ((int)blockIdx.x >= pack_blocks) {
    transpose_grids_tile(grids, m, blockIdx.x - pack_blocks);
    return;
  }
  const int chunks = n / kChunk;
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= (int64_t)m * chunks) return;
  const int c = (int)(e / m), row = (int)(e - (int64_t)c * m);   // rows fastest: the stores are contiguous
  const uint4* src = reinterpret_cast<const uint4*>(codes + (int64_t)row * ldc + c * kChunk);
  const uint4 lo = src[0], hi = src[1];
  const uint32_t raw[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
  uint32_t* dst = packed + ((int64_t)c * m + row) * BITS;
  uint64_t acc = 0;
  int have = 0, w = 0;
#pragma unroll
  for (int j = 0; j < kChunk; ++j) {
    const uint32_t code = (raw[j >> 2] >> (8 * (j & 3))) & ((1u << BITS) - 1u);
    acc |= (uint64_t)code << have;
    have += BITS;
    if (have >= 32) {
      dst[w++] = (uint32_t)acc;
      acc >>= 32;
      have -= 32;
    }
  }
}

template <int BITS>
__global__ __launch_bounds__(256) void unpack_dequant_kernel(const uint32_t* __restrict__ packed, int m, int n,
                                                             const float* __restrict__ scales,
                                                             const uint8_t* __restrict__ zeros, int group,
                                                             double* __restrict__ Wq, int64_t ldq) {
  const int chunks = n / kChunk;
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= (int64_t)m * chunks) return;
  const int c = (int)(e / m), row = (int)(e - (int64_t)c * m);
  const uint32_t* src = packed + ((int64_t)c * m + row) * BITS;
  uint32_t words[BITS];
#pragma unroll
  for (int w = 0; w < BITS; ++w) words[w] = src[w];
  uint8_t code[kChunk];
  unpack_chunk<BITS>(words, code);
  double* dst = Wq + (int64_t)row * ldq + c * kChunk;
#pragma unroll
  for (int j = 0; j < kChunk; ++j) {
    const int g = (c * kChunk + j) / group;   // a group may be as small as 16 columns
    const double sc = (double)scales[(int64_t)g * m + row];
    const double z = (double)zeros[(int64_t)g * m + row];
    dst[j] = sc * ((double)code[j] - z);
  }
}

// ---- the layer applied to tokens ------------------------------------------------------------
__device__ __forceinline__ float e4m3_to_float(uint8_t c) {
  // exponent and mantissa in place of a float32's, subnormals included; 2^120 = the difference of the biases
  const float mag = __uint_as_float((uint32_t)(c & 0x7f) << 20) * 0x1p120f;
  return __uint_as_float(__float_as_uint(mag) | (uint32_t)(c & 0x80) << 24);
}
__device__ __forceinline__ float fp16_bits_to_float(uint16_t h) {
  const int ef = (h >> 10) & 31, mt = h & 0x3ff;
  float mag;
  if (ef == 31) mag = mt ? __builtin_nanf("") : __builtin_inff();
  else mag = ef == 0 ? ldexpf((float)mt, -24) : ldexpf((float)(1024 + mt), ef - 25);
  return (h & 0x8000) ? -mag : mag;
}

// ---- what the products read: X~ and the low-rank coefficients, one launch -------------------------
// X~ = X P Q in float64, written as float32 (xt[chunk][token][32]) for the few-token product, as two float16 pieces
// ([2][32] in the same place) for the tiles (but for tokens that these do not hold), and, in float64,
//   y[t][k] = sigma_k * sum_j V[k][j] x[t][j] / s[j].
// The first workgroups take y: a token and four ranks each, or 16 tokens x 16 ranks on the float64 matrix instruction from
// kPrepMany tokens on.  The others rotate: a workgroup stages the rows of a token (several, where they are narrow and many)
// in LDS and transforms 256-column chunks, a wave each (a row goes to several workgroups while there are few tokens).
// For a few tokens both parts are chains of latencies; for many the rotation is vector instructions (some 200 per
// chunk).  512 tokens x 11008 columns, 16 ranks: 30 us as float32 with 2 tokens x 16 ranks of y per workgroup on the vector
// unit (the rotation alone 15), now 26 with the pieces and the look at each token's small entries (24 without it); 4000 x 1024 34 -> 22.
struct PrepArgs {
  const void* X;
  int64_t ldx;
  int tokens, n;
  const int32_t* perm;
  int b_I;
  const uint8_t* V;
  const uint16_t* sigma;
  const double* s;
  int r;
  float* xt;
  float* y;
  double* y_parts;      // null: y; else coeff_splits x tokens x r, without sigma
  int coeff_tiles, coeff_splits;
  int run_lg, segments, segment;   // 2^run_lg tokens a rotating workgroup; workgroups per token (run_lg = 0) and chunks of each
  uint64_t order;   // 0: X~ as float32; otherwise as two float16 pieces, position p of 16 holds column (order >> 4 p) & 15
  int* exponents;   // tokens: X~ is 2^exponents[token] times the pieces' sum; kPlain: X~ as float32
  bool roomy;       // LDS beyond the row: kPrepExtra bytes
  int lg;           // b_H = 2^lg
  double scale;     // 1 / sqrt(b_H)
};

constexpr int kPrepThreads = 512, kPrepWaves = kPrepThreads / 64;
constexpr int kPrepExtra = kPrepWaves * (2 + 256) * (int)sizeof(uint32_t);
constexpr int kPlain = INT_MIN;
// From here on 16 tokens share a wave's quotients and conversions (whole call, 16 ranks: 200 x 4096 x 11008 75 us, 76 without;
// 512 x 4096 x 11008 120 and 139; 1000 x 777 x 512 27 and 37).  Below it the chip is not full that way (128 x 4096 x 11008 57
// and 52 us, 160 x 11008 x 4096 91 and 87).
constexpr int kPrepMany = 192;   // tokens
constexpr int kCoeffSplits = 4;  // workgroups that share the columns of 16 tokens x 16 ranks

// Sums of NV values per lane over the 64 lanes, halving the number of values with every exchange as long as there
// is more than one: afterwards v[0] is the sum of value (lane / (64 / NV)).
template <int NV, int MASK>
__device__ __forceinline__ void fold_lanes(double* v, int lane) {
  if constexpr (MASK > 0) {
    constexpr int H = NV > 1 ? NV / 2 : 1;
    const bool upper = lane & MASK;
#pragma unroll
    for (int i = 0; i < H; ++i) {
      const double a = v[i], b = NV > 1 ? v[i + H] : v[i];
      if constexpr (MASK >= 16) {
        double first, second;
        lane_pair<MASK == 32>(a, b, first, second);
        v[i] = first + second;
      } else {
        const double keep = upper ? b : a, send = upper ? a : b;
        double got;
        if constexpr (MASK == 8) got = dpp_move<kDppRotate8>(send);
        else if constexpr (MASK == 4) got = dpp_move<kDppReverseQuad>(dpp_move<kDppHalfMirror>(send));
        else if constexpr (MASK == 2) got = dpp_move<kDppSwapHalfQuads>(send);
        else got = dpp_move<kDppSwapPairs>(send);
        v[i] = keep + got;
      }
    }
    fold_lanes<H, MASK / 2>(v, lane);
  }
}

template <int DT, bool ALIGNED, int TG, int RG>
__device__ __forceinline__ void low_rank_coefficients(const PrepArgs& a, double* red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int rank_tiles = (a.r + RG - 1) / RG;
  const int t0 = (blockIdx.x / rank_tiles) * TG, k0 = (blockIdx.x % rank_tiles) * RG;
  using ST = typename StoredType<DT>::type;
  const ST* xp[TG];   // tokens and ranks past the end repeat the last; not stored
#pragma unroll
  for (int t = 0; t < TG; ++t) xp[t] = static_cast<const ST*>(a.X) + (int64_t)min(t0 + t, a.tokens - 1) * a.ldx;
  const uint8_t* vp[RG];
#pragma unroll
  for (int k = 0; k < RG; ++k) vp[k] = a.V + (int64_t)min(k0 + k, a.r - 1) * a.n;
  double acc[TG * RG];
#pragma unroll
  for (int i = 0; i < TG * RG; ++i) acc[i] = 0.0;
  for (int j = 4 * threadIdx.x; j < a.n; j += 4 * kPrepThreads) {
    struct alignas(ALIGNED ? 4 * sizeof(ST) : sizeof(ST)) Quad { ST e[4]; };
    struct alignas(ALIGNED ? 16 : 8) Scale { double e[4]; };
    struct alignas(ALIGNED ? 4 : 1) Codes { uint8_t e[4]; };
    Quad x[TG];
    Codes c[RG];
    const Scale sc = *reinterpret_cast<const Scale*>(a.s + j);
#pragma unroll
    for (int t = 0; t < TG; ++t) x[t] = *reinterpret_cast<const Quad*>(xp[t] + j);
#pragma unroll
    for (int k = 0; k < RG; ++k) c[k] = *reinterpret_cast<const Codes*>(vp[k] + j);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      double xs[TG];
#pragma unroll
      for (int t = 0; t < TG; ++t) xs[t] = stored_to_f64<DT>(x[t].e[i]) / sc.e[i];
#pragma unroll
      for (int k = 0; k < RG; ++k) {
        const double v = (double)e4m3_to_float(c[k].e[i]);
#pragma unroll
        for (int t = 0; t < TG; ++t) acc[t * RG + k] = fma(v, xs[t], acc[t * RG + k]);
      }
    }
  }
  constexpr int NV = TG * RG;
  fold_lanes<NV, 32>(acc, lane);
  if (lane % (64 / NV) == 0) red[wave * NV + lane / (64 / NV)] = acc[0];
  __syncthreads();
  if (threadIdx.x < NV) {
    double sum = 0.0;
#pragma unroll
    for (int w = 0; w < kPrepWaves; ++w) sum += red[w * NV + threadIdx.x];
    const int t = t0 + (int)threadIdx.x / RG, k = k0 + (int)threadIdx.x % RG;
    if (t < a.tokens && k < a.r) a.y[(int64_t)t * a.r + k] = (float)(sum * (double)fp16_bits_to_float(a.sigma[k]));
  }
}

__device__ __host__ __forceinline__ int align16(int bytes) { return (bytes + 15) & ~15; }

// low halves of two words, the lower one first, and their high halves
__device__ __forceinline__ uint32_t pair_low(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); }
__device__ __forceinline__ uint32_t pair_high(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }

// A number below 2^15 as the sum of a float16 and 2^-kSecond of another: each rounded to nearest, the second of what the
// first leaves, which is at most 2^3
constexpr int kSecond = 12;
__device__ __forceinline__ uint32_t split2(double x) {
  // by way of float32, kept apart: as one conversion from float64 it is some forty instructions
  auto narrow = [](double v) {
    float f = (float)v;
    asm("" : "+v"(f));
    return (_Float16)f;
  };
  const _Float16 first = narrow(x);
  const _Float16 second = narrow((x - (double)first) * (double)(1 << kSecond));
  return (uint32_t)__builtin_bit_cast(uint16_t, second) << 16 | __builtin_bit_cast(uint16_t, first);
}

// Many tokens: 16 of them x 16 ranks on the float64 matrix instruction, the columns dealt to the waves of coeff_splits
// workgroups, 32 at a time: lane l is token (rank) l % 16 and takes columns 8 (l / 16) .. + 7.  A column's reciprocal
// 1 / s serves all tokens; the quotient x / s it gives is corrected by its remainder, x - q s being exact, and
// is right to an ulp of float64.  Where that fails (x infinite, s beyond 2^500 or below 2^-500) the remainder is NaN, and the
// division itself is done.
template <int DT, bool ALIGNED>
__device__ __forceinline__ void low_rank_coefficients_many(const PrepArgs& a, char* lds) {
  using ST = typename StoredType<DT>::type;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = (lane >> 4) * 8;
  const int rank_tiles = (a.r + 15) / 16;
  const int split = blockIdx.x % a.coeff_splits, tile = blockIdx.x / a.coeff_splits;
  const int t0 = (tile / rank_tiles) * 16, k0 = (tile % rank_tiles) * 16;
  // tokens and ranks past the end repeat the last; not stored
  const ST* xp = static_cast<const ST*>(a.X) + (int64_t)min(t0 + (lane & 15), a.tokens - 1) * a.ldx + col;
  const uint8_t* vp = a.V + (int64_t)min(k0 + (lane & 15), a.r - 1) * a.n + col;
  struct Column { double s, inverse; };
  Column* table = reinterpret_cast<Column*>(lds) + 32 * wave;
  struct alignas(ALIGNED ? 16 : sizeof(ST)) Eight { ST e[8]; };
  struct alignas(ALIGNED ? 4 : 1) Codes { uint8_t e[8]; };
  f64x4 acc = {0.0, 0.0, 0.0, 0.0};
  const int blocks = a.n / 32, stride = kPrepWaves * a.coeff_splits;
  int b = split * kPrepWaves + wave;
  Eight x;
  Codes c;
  double sv = 1.0;
  auto request = [&](int at) {
    at = min(at, blocks - 1) * 32;   // issued whatever the block: no branch
    x = *reinterpret_cast<const Eight*>(xp + at);
    c = *reinterpret_cast<const Codes*>(vp + at);
    sv = a.s[at + (lane & 31)];
  };
  request(b);
  for (; b < blocks; b += stride) {
    const double mag = fabs(sv);
    const bool safe = DT != PTQ_F64 && mag > 0x1p-500 && mag < 0x1p500;
    table[lane & 31] = Column{sv, safe ? 1.0 / sv : __builtin_nan("")};
    __builtin_amdgcn_wave_barrier();
    const Eight xb = x;
    const Codes cb = c;
    request(b + stride);
    double q[8], v[8], sum = 0.0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const Column t = table[col + i];
      const double xv = stored_to_f64<DT>(xb.e[i]), q0 = xv * t.inverse;
      q[i] = fma(fma(-q0, t.s, xv), t.inverse, q0);
      sum += q[i];
    }
    if (__builtin_isnan(sum)) {
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (__builtin_isnan(q[i])) q[i] = stored_to_f64<DT>(xb.e[i]) / table[col + i].s;
    }
#pragma unroll
    for (int i = 0; i < 8; i += 2) {   // e4m3 in place of a float16's upper bits: 2^-8 of its value
      const uint32_t two = (uint32_t)cb.e[i] | (uint32_t)cb.e[i + 1] << 16;
      const uint32_t h = (two & 0x007f007fu) << 7 | (two & 0x00800080u) << 8;
      typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
      const f16x2 f = __builtin_bit_cast(f16x2, h);
      v[i] = (double)(float)f.x;
      v[i + 1] = (double)(float)f.y;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(q[i], v[i], acc, 0, 0, 0);
    __builtin_amdgcn_wave_barrier();
  }
  // accumulator k of a lane is token 4 k + lane / 16, rank lane % 16; the waves' sums in order
  __syncthreads();
  double* red = reinterpret_cast<double*>(lds);
#pragma unroll
  for (int k = 0; k < 4; ++k) red[wave * 256 + k * 64 + lane] = acc[k];
  __syncthreads();
  if (threadIdx.x < 256) {
    double sum = 0.0;
#pragma unroll
    for (int w = 0; w < kPrepWaves; ++w) sum += red[w * 256 + threadIdx.x];
    sum *= 0x1p8;
    const int t = t0 + 4 * wave + (lane >> 4), k = k0 + (lane & 15);
    if (t < a.tokens && k < a.r) {
      if (a.y_parts) a.y_parts[((int64_t)split * a.tokens + t) * a.r + k] = sum;
      else a.y[(int64_t)t * a.r + k] = (float)(sum * (double)fp16_bits_to_float(a.sigma[k]));
    }
  }
}

// the part of a stored number that orders magnitudes: float32 bits, the upper half of a float64
template <int DT>
__device__ __forceinline__ uint32_t magnitude(typename StoredType<DT>::type v) {
  if constexpr (DT == PTQ_F64) return (uint32_t)((uint64_t)__double_as_longlong(v) >> 32) & 0x7fffffffu;
  else if constexpr (DT == PTQ_F32) return __float_as_uint(v) & 0x7fffffffu;
  else return ((uint32_t)v << 16) & 0x7fffffffu;
}

// ... and powers of two among them
template <int DT>
struct Magnitudes {
  static constexpr int kMantissa = DT == PTQ_F64 ? 20 : 23, kBias = DT == PTQ_F64 ? 1023 : 127;
  static __device__ bool finite(uint32_t v) { return (int)(v >> kMantissa) != 2 * kBias + 1; }
  static __device__ int exponent(uint32_t v) {   // 2^exponent <= v < 2^(exponent + 1); v > 0
    const int field = (int)(v >> kMantissa);
    return field ? field - kBias : 31 - __clz((int)v) - kMantissa - (kBias - 1);
  }
  static __device__ uint32_t power(int e) {   // 2^e, at most the largest; 0 below the smallest
    return e > -kBias ? (uint32_t)(e + kBias) << kMantissa : (e + kBias - 1 + kMantissa >= 0 ? 1u << (e + kBias - 1 + kMantissa) : 0u);
  }
};

__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
  auto with = [&](auto ctrl) { v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, decltype(ctrl)::value, 0xf, 0xf, false)); };
  with(std::integral_constant<int, kDppSwapPairs>{});
  with(std::integral_constant<int, kDppSwapHalfQuads>{});
  with(std::integral_constant<int, kDppHalfMirror>{});
  with(std::integral_constant<int, kDppMirror>{});
  const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)v, 0), b = (uint32_t)__builtin_amdgcn_readlane((int)v, 16);
  const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)v, 32), d = (uint32_t)__builtin_amdgcn_readlane((int)v, 48);
  return max(max(a, b), max(c, d));
}

template <int DT, bool ALIGNED, bool PIECES>
__global__ __launch_bounds__(kPrepThreads, 4) void forward_prep_kernel(PrepArgs a) {
  extern __shared__ __attribute__((aligned(16))) char prep_lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = (int)__builtin_amdgcn_readfirstlane(tid >> 6);
  // all arguments at once: fetched where they are used they are a chain of trips to memory (with those of the product for a few
  // tokens, 2 x 4096 x 4096 14.4 -> 13.8 us, 3 x 4096 x 4096 17.1 -> 16.6; the forms with pieces spill 52 scalar registers for it and are no slower)
  asm volatile("" ::"s"(a.X), "s"(a.ldx), "s"(a.tokens), "s"(a.n), "s"(a.perm), "s"(a.b_I), "s"(a.xt), "s"(a.run_lg), "s"(a.segments),
               "s"(a.segment), "s"(a.order), "s"((int)a.roomy), "s"(a.lg), "s"(a.scale), "s"(a.V), "s"(a.s), "s"(a.r), "s"(a.y), "s"(a.coeff_tiles));
  if ((int)blockIdx.x < a.coeff_tiles) {
    if (PIECES && a.tokens >= kPrepMany) low_rank_coefficients_many<DT, ALIGNED>(a, prep_lds);
    else low_rank_coefficients<DT, ALIGNED, 1, 4>(a, reinterpret_cast<double*>(prep_lds));
    return;
  }
  using ST = typename StoredType<DT>::type;
  const int item = blockIdx.x - a.coeff_tiles, run_lg = a.run_lg;
  const int unit = a.segments == 1 ? item : item / a.segments;
  const int token0 = unit << run_lg, seg = item - unit * a.segments;
  const int run = min(1 << run_lg, a.tokens - token0);
  const int row = align16(a.n * (int)sizeof(ST));
  // A wave stages a share of one token's row and keeps its largest magnitude, a lane of its entries the smallest but zero, less one
  const int my = wave & ((1 << run_lg) - 1), shares = kPrepWaves >> run_lg;
  uint32_t top = 0, bottom = ~0u;
  if (my < run) {
    const ST* src = static_cast<const ST*>(a.X) + (int64_t)(token0 + my) * a.ldx;
    ST* dst = reinterpret_cast<ST*>(prep_lds + my * row);
    constexpr int kPer = ALIGNED ? 16 / (int)sizeof(ST) : 1;   // n is a multiple of 32
    struct alignas(ALIGNED ? 16 : sizeof(ST)) Piece { ST e[kPer]; };
    for (int c = ((wave >> run_lg) * 64 + lane) * kPer; c < a.n; c += shares * 64 * kPer) {
      const Piece p = *reinterpret_cast<const Piece*>(src + c);
      *reinterpret_cast<Piece*>(dst + c) = p;
      if constexpr (PIECES) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
          const uint32_t v = magnitude<DT>(p.e[i]);
          top = max(top, v);
          bottom = min(bottom, v - 1);
        }
      }
    }
  }
  uint32_t* tops = reinterpret_cast<uint32_t*>(prep_lds + (row << run_lg));   // with pieces and where there is room: of each wave
  uint32_t* swap = tops + 2 * kPrepWaves + 256 * wave;                        // ... and a wave's own 256 words
  if (PIECES && a.roomy) {
    top = wave_max(top);
    if (lane == 0) tops[wave] = top;
  }
  const int nchunk_id = (a.b_I + 255) / 256;                   // chunks of the identity part
  const int nchunk = nchunk_id + (a.n - a.b_I + 255) / 256;    // ... plus those of the rotated part
  const int lg = a.lg;
  const int k_begin = seg * a.segment, items = (min(nchunk, k_begin + a.segment) - k_begin) << run_lg;
  // item i: token i % 2^run_lg of chunk k_begin + i / 2^run_lg, its columns first .. first + 255 as far as they lie below `end`
  struct Chunk { int first, end; bool rotated; };
  auto chunk_of = [&](int i) {
    const int k = k_begin + (i >> run_lg);
    const bool rotated = k >= nchunk_id;
    return Chunk{rotated ? a.b_I + 256 * (k - nchunk_id) : 256 * k, rotated ? a.n : a.b_I, rotated};
  };
  auto places = [&](int i) {
    return *reinterpret_cast<const int4*>(a.perm + min(chunk_of(i).first + 4 * lane, a.n - 4));
  };
  int4 next = places(min(wave, items - 1));
  __syncthreads();
  // X~ 2^up stays below 2^15: 2^e <= max |x| < 2^(e + 1) (rows of zeros and rows with an infinity or a NaN, whose outputs are
  // NaN, go as they are), and a rotation makes it sqrt(b_H) times as large at most.  Lane tl holds token tl's.
  // The pieces hold 23 bits of what is no smaller than 2^-kSpan of the largest, and 2^-47 of the largest of anything.  That is
  // below the rounding of the float32 sums unless most of what a row sees is smaller: a token with more than a quarter of its entries
  // below the line goes as float32, and the product takes it by itself, at some eighteen times the cost (64 x 4096 x 700: 24 us, 425 with
  // all tokens of that kind; entries up to 2^22 times the others stay).  Most tokens of heavy-tailed activations have such
  // entries, but few: only the lanes that have staged one look at theirs again.
  int ups = 0;
  uint32_t from[4];   // where a lane's four positions of 16 come from
  if constexpr (PIECES) {
    using M = Magnitudes<DT>;
    constexpr int kSpan = 24;
    const auto of_token = [&](int w) { return ((w ^ lane) & ((1 << run_lg) - 1)) == 0; };   // wave w's share and lane's token
    static_assert(kPrepWaves == 8, "two reads");
    const auto read8 = [&](int at, auto f) {   // the waves' words
      const uint4 lo = reinterpret_cast<const uint4*>(tops + at)[0], hi = reinterpret_cast<const uint4*>(tops + at)[1];
      const uint32_t t[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
      for (int w = 0; w < 8; ++w) f(of_token(w) ? t[w] : 0u);
    };
    uint32_t largest = 0;
    if (a.roomy) {
      read8(0, [&](uint32_t v) { largest = max(largest, v); });
    } else {   // one row
      for (int q = lane; q < a.n; q += 64) largest = max(largest, magnitude<DT>(reinterpret_cast<const ST*>(prep_lds)[q]));
      largest = wave_max(largest);
    }
    const bool ordinary = largest != 0 && M::finite(largest);
    const int e = ordinary ? M::exponent(largest) : 0;
    ups = ordinary ? min(14 - e - (lg + 1) / 2, 1000) : 0;
    const uint32_t limit = ordinary ? M::power(e - kSpan) : 0u, below = limit ? limit - 1 : 0u;   // v - 1 < below: 0 < v < limit
    const uint32_t mine = a.roomy ? (uint32_t)__builtin_amdgcn_readlane((int)below, my) : below;
    int count = 0;
    if (!a.roomy) {
      for (int q = lane; q < a.n; q += 64) count += magnitude<DT>(reinterpret_cast<const ST*>(prep_lds)[q]) - 1 < mine;
    } else if (bottom < mine) {
      constexpr int kPer = ALIGNED ? 16 / (int)sizeof(ST) : 1;
      const ST* src = reinterpret_cast<const ST*>(prep_lds + my * row);
      for (int c = ((wave >> run_lg) * 64 + lane) * kPer; c < a.n; c += shares * 64 * kPer)
        for (int i = 0; i < kPer; ++i) count += magnitude<DT>(src[c + i]) - 1 < mine;
    }
    if (__ballot(count > 0)) {
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) count += __shfl_xor(count, off);
    }
    if (a.roomy) {
      if (lane == 0) tops[kPrepWaves + wave] = (uint32_t)count;
      __syncthreads();
      count = 0;
      read8(kPrepWaves, [&](uint32_t v) { count += (int)v; });
    }
    if (count > a.n / 4) ups = kPlain;
    if (seg == 0 && tid < run) a.exponents[token0 + tid] = ups == kPlain ? kPlain : -ups;
    const uint32_t order = (uint32_t)(a.order >> (16 * (lane & 3)));
#pragma unroll
    for (int q = 0; q < 4; ++q) from[q] = 4 * (lane & ~3) + ((order >> (4 * q)) & 15);
  }
  for (int i = wave; i < items; i += kPrepWaves) {
    const int tl = i & ((1 << run_lg) - 1), token = token0 + tl;
    const Chunk ch = chunk_of(i);
    const int4 p = next;
    if (i + kPrepWaves < items) next = places(i + kPrepWaves);
    if (tl >= run) continue;
    const int c = ch.first + 4 * lane;
    const bool live = c < ch.end;
    const ST* buf = reinterpret_cast<const ST*>(prep_lds + tl * row);
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    if (live) {
      v[0] = stored_to_f64<DT>(buf[p.x]);
      v[1] = stored_to_f64<DT>(buf[p.y]);
      v[2] = stored_to_f64<DT>(buf[p.z]);
      v[3] = stored_to_f64<DT>(buf[p.w]);
    }
    if (ch.rotated) fwht_chunk(v, lg, lane);
    const int up = PIECES ? __builtin_amdgcn_readlane(ups, tl) : kPlain;
    if (PIECES || ch.rotated) {
      const double factor = ch.rotated ? a.scale : 1.0, unit = up != kPlain ? ldexp(factor, up) : factor;
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] *= unit;
    }
    // of the token's 128 bytes in each of the 32-column pieces c / 32; c is a multiple of 4
    char* const base = reinterpret_cast<char*>(a.xt) + (int64_t)token * (kChunk * 4);
    const uint32_t at = (uint32_t)(c >> 5) * ((uint32_t)a.tokens * (kChunk * 4));
    if (!PIECES || up == kPlain) {
      if (live) *reinterpret_cast<float4*>(base + (at + 4 * (c & 31))) = make_float4((float)v[0], (float)v[1], (float)v[2], (float)v[3]);
      continue;
    }
    uint32_t both[4];   // the second piece above the first
#pragma unroll
    for (int q = 0; q < 4; ++q) both[q] = split2(v[q]);
    if (a.roomy) {   // a group of 16 columns is whole: b_I and n are multiples of 16
      *reinterpret_cast<uint4*>(swap + 4 * lane) = make_uint4(both[0], both[1], both[2], both[3]);
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int q = 0; q < 4; ++q) both[q] = swap[from[q]];
      __builtin_amdgcn_wave_barrier();
      if (live) {
        char* dst = base + (at + 2 * (c & 31));
        *reinterpret_cast<uint2*>(dst) = make_uint2(pair_low(both[0], both[1]), pair_low(both[2], both[3]));
        *reinterpret_cast<uint2*>(dst + 2 * kChunk) = make_uint2(pair_high(both[0], both[1]), pair_high(both[2], both[3]));
      }
    } else if (live) {
      for (int q = 0; q < 16; ++q) {
        const int j = (int)(a.order >> (4 * q)) & 15;
        if ((j >> 2) != (lane & 3)) continue;
        const uint32_t w = (j & 2) ? ((j & 1) ? both[3] : both[2]) : ((j & 1) ? both[1] : both[0]);
        uint16_t* dst = reinterpret_cast<uint16_t*>(base + at) + (c & 16) + q;
        dst[0] = (uint16_t)w;
        dst[kChunk] = (uint16_t)(w >> 16);
      }
    }
  }
}

template <int DT>
ptq_status launch_forward_prep(PrepArgs a, hipStream_t st) {
  using ST = typename StoredType<DT>::type;
  const size_t row = (size_t)a.n * sizeof(ST);
  if (row > 160 * 1024) return PTQ_ERR_SHAPE;
  const int nchunk = (a.b_I + 255) / 256 + (a.n - a.b_I + 255) / 256;
  const bool many = a.tokens >= kPrepMany;
  a.coeff_tiles = (int)(many ? ceil_div(a.tokens, 16) * ceil_div(a.r, 16) * a.coeff_splits : a.tokens * ceil_div(a.r, 4));
  // every workgroup of a token stages its whole row: split it only as far as that fills the chip.  Narrow rows of many
  // tokens go several to a workgroup, until its waves have two chunks each.
  a.segments = (int)std::min<int64_t>(ceil_div(nchunk, kPrepWaves), ceil_div(256, a.tokens));
  a.segment = (int)ceil_div(nchunk, a.segments);
  a.run_lg = 0;
  while (a.run_lg < 3 && a.segments == 1 && (nchunk << a.run_lg) < 2 * kPrepWaves && a.tokens >> (a.run_lg + 1) >= 512 &&
         2 * row << a.run_lg <= 32 * 1024)
    ++a.run_lg;
  const size_t rows = (size_t)align16((int)row) << a.run_lg;
  a.roomy = rows + kPrepExtra <= 160 * 1024;
  const auto off = [](const void* p) { return reinterpret_cast<uintptr_t>(p) % 16; };
  const bool aligned = off(a.X) == 0 && (a.ldx * sizeof(ST)) % 16 == 0 && (a.r == 0 || (off(a.V) % 4 == 0 && off(a.s) == 0));
  const size_t coeff = many ? (size_t)kPrepWaves * 256 * sizeof(double) : (size_t)kPrepWaves * 4 * sizeof(double);
  const size_t lds = std::max(a.order && a.roomy ? rows + kPrepExtra : std::max(rows, row), a.r ? coeff : 0);
  const unsigned grid = (unsigned)(a.coeff_tiles + ceil_div(a.tokens, (int64_t)1 << a.run_lg) * a.segments);
  const auto launch = [&](auto is_aligned, auto pieces) {
    constexpr auto kernel = forward_prep_kernel<DT, decltype(is_aligned)::value, decltype(pieces)::value>;
    if (!lds_opt_in<kernel>(160 * 1024)) return PTQ_ERR_HIP;
    kernel<<<grid, kPrepThreads, lds, st>>>(a);
    return PTQ_OK;
  };
  if (a.order) return aligned ? launch(std::true_type{}, std::true_type{}) : launch(std::false_type{}, std::true_type{});
  return aligned ? launch(std::true_type{}, std::false_type{}) : launch(std::false_type{}, std::false_type{});
}

struct ForwardArgs {
  const uint32_t* packed;   // (n / 32) x m x BITS words
  const float* scales;      // n / group x m
  const uint8_t* zeros;     // n / group x m
  int m, n, group;
  const float* xt;          // X~, 32 columns of all tokens at a time: xt[chunk][token][32], or two float16 pieces [2][32] in its place
  int xt_tokens;            // tokens per chunk of xt
  const float* y;           // tokens x r
  const double* y_parts;    // null: y; else y_splits x tokens x r, to be added and multiplied by sigma
  int y_splits;
  const uint16_t* sigma;
  const uint8_t* U;         // r x m, e4m3
  int r;
  const int* exponents;     // tokens: with pieces, X~ is 2^exponent times their sum; kPlain: X~ as float32
  float* partial;           // (splits - 1) x tokens x m: the first split's sums go to O
  float* O;                 // tokens x m
  int64_t ldo;
};

// ---- a few tokens ----------------------------------------------------------------------------
// Bound by the codes' way from memory.  A lane is a row (R consecutive ones per workgroup) and a slice of the
// columns: the 256 / R slices of a workgroup take every (256 / R)-th chunk, eight at a time (their words are
// requested before anything else), X~ of all columns sits in LDS (a slice's lanes read the same address), and the
// slices are added by lane exchanges and through LDS -- no partial sums in memory and no counting of
// workgroups.  sum_j scale (code_j - zero) x_j = scale (sum_j code_j x_j - zero sum_j x_j): the second sum does not
// depend on the row, so a weight costs a conversion and a multiply-add per token (half an instruction to
// extract).  The ranks of the low-rank part are dealt to the slices like chunks.  One token, 4096 x 4096, 4 bits:
// 7.6 us for the kernel (11.8 with a workgroup per 256 rows x 256 columns, partial sums in memory and the last
// workgroup of a row block adding them); 16 rows per workgroup, 8 where that leaves compute units idle.
template <int BITS>
struct alignas(BITS == 3 ? 4 : (BITS == 2 ? 8 : 16)) Words { uint32_t w[BITS]; };

// codes [8 Q, 8 Q + 8) of a chunk
template <int BITS, int Q>
__device__ __forceinline__ void codes_to_float(const Words<BITS>& v, float (&f)[8]) {
  if constexpr (BITS == 8) {
#pragma unroll
    for (int j = 0; j < 8; ++j) f[j] = (float)((v.w[2 * Q + (j >> 2)] >> (8 * (j & 3))) & 0xffu);
  } else if constexpr (BITS == 4) {
    const uint32_t even = v.w[Q] & 0x0f0f0f0fu, odd = (v.w[Q] >> 4) & 0x0f0f0f0fu;
#pragma unroll
    for (int j = 0; j < 8; ++j) f[j] = (float)((((j & 1) ? odd : even) >> (8 * (j >> 1))) & 0xffu);
  } else if constexpr (BITS == 2) {
#pragma unroll
    for (int j = 0; j < 8; ++j)
      f[j] = (float)((((v.w[Q >> 1] >> (16 * (Q & 1) + 2 * (j & 3))) & 0x0303u) >> (8 * (j >> 2))) & 0xffu);
  } else {
    constexpr int pos = 24 * Q, wi = pos >> 5, sh = pos & 31;
    uint32_t b = v.w[wi] >> sh;
    if constexpr (sh + 24 > 32) b |= v.w[wi + 1] << (32 - sh);
#pragma unroll
    for (int j = 0; j < 8; ++j) f[j] = (float)((b >> (3 * j)) & 7u);
  }
}

constexpr int kRowBatch = 8;             // chunks per lane on their way at a time
constexpr int kRowLdsFloats = 36 * 1024;  // X~ staged at a time: columns x tokens, plus 1/32 of it for the chunk sums

// B tokens, rows [R q, R q + R) of the weight for item q; `columns` (a multiple of 32) are staged at a time
template <int BITS, int B, int R>
__global__ __launch_bounds__(256) void forward_rows_kernel(ForwardArgs a, int columns, int items) {
  extern __shared__ __attribute__((aligned(16))) float row_lds[];
  constexpr int S = 256 / R;
  // all arguments at once, not one after the other where they are used
  asm volatile("" ::"s"(a.packed), "s"(a.scales), "s"(a.zeros), "s"(a.m), "s"(a.n), "s"(a.group), "s"(a.xt), "s"(a.xt_tokens), "s"(a.y),
               "s"(a.U), "s"(a.r), "s"(a.O), "s"(a.ldo), "s"(columns), "s"(items));
  const int per = (items + 7) / 8;   // consecutive items on one XCD: neighbouring rows share cache lines
  const int q = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per || q >= items) return;
  const int tid = threadIdx.x, lane = tid & 63, slice = tid / R;
  const int m = a.m, chunks = a.n / kChunk;
  const int row = q * R + tid % R;
  const int64_t rr = min(row, m - 1);   // a lane past the last row repeats it; not stored
  const uint32_t* packed = a.packed + rr * BITS;
  const int stage = columns / kChunk;
  float* xs = row_lds;                    // [B][columns]
  float* xsum = row_lds + B * columns;    // [B][stage]
  float acc[B];
#pragma unroll
  for (int t = 0; t < B; ++t) acc[t] = 0.f;
  for (int c0 = 0; c0 < chunks; c0 += stage) {
    const int nc = min(stage, chunks - c0);
    Words<BITS> wd[kRowBatch];
    float sc[kRowBatch], zero[kRowBatch];
    auto request = [&](int i0) {
#pragma unroll
      for (int i = 0; i < kRowBatch; ++i) {
        const int c = c0 + min(i0 + i * S + slice, nc - 1);   // issued whatever the chunk: no branch
        wd[i] = *reinterpret_cast<const Words<BITS>*>(packed + (int64_t)c * m * BITS);
        const int64_t g = c * kChunk / a.group;
        sc[i] = a.scales[g * m + rr];
        zero[i] = (float)a.zeros[g * m + rr];
      }
    };
    request(0);
    if (c0 > 0) __syncthreads();
    for (int e = tid; e < B * nc * (kChunk / 4); e += 256) {   // eight consecutive threads hold one chunk
      const int t = e / (nc * (kChunk / 4)), k = e - t * (nc * (kChunk / 4));
      const float4 v = *reinterpret_cast<const float4*>(a.xt + ((int64_t)(c0 + (k >> 3)) * a.xt_tokens + t) * kChunk + 4 * (k & 7));
      *reinterpret_cast<float4*>(xs + t * columns + 4 * k) = v;
      float sum = (v.x + v.y) + (v.z + v.w);
      sum += __shfl_xor(sum, 1);
      sum += __shfl_xor(sum, 2);
      sum += __shfl_xor(sum, 4);
      if ((k & 7) == 0) xsum[t * stage + (k >> 3)] = sum;
    }
    __syncthreads();
    for (int i0 = 0; i0 < nc; i0 += kRowBatch * S) {
      if (i0 > 0) request(i0);
#pragma unroll
      for (int i = 0; i < kRowBatch; ++i) {
        const int c = i0 + i * S + slice;
        const int cl = min(c, nc - 1);
        float raw[B];
#pragma unroll
        for (int t = 0; t < B; ++t) raw[t] = 0.f;
        auto eight = [&](auto quarter) {
          constexpr int Q = decltype(quarter)::value;
          float f[8];
          codes_to_float<BITS, Q>(wd[i], f);
#pragma unroll
          for (int t = 0; t < B; ++t) {
            const float4* x = reinterpret_cast<const float4*>(xs + t * columns + cl * kChunk + 8 * Q);
            const float4 lo = x[0], hi = x[1];
            raw[t] = fmaf(f[3], lo.w, fmaf(f[2], lo.z, fmaf(f[1], lo.y, fmaf(f[0], lo.x, raw[t]))));
            raw[t] = fmaf(f[7], hi.w, fmaf(f[6], hi.z, fmaf(f[5], hi.y, fmaf(f[4], hi.x, raw[t]))));
          }
        };
        eight(std::integral_constant<int, 0>{});
        eight(std::integral_constant<int, 1>{});
        eight(std::integral_constant<int, 2>{});
        eight(std::integral_constant<int, 3>{});
        if (c < nc) {
#pragma unroll
          for (int t = 0; t < B; ++t) acc[t] = fmaf(sc[i], fmaf(-zero[i], xsum[t * stage + cl], raw[t]), acc[t]);
        }
      }
    }
  }
  for (int k = slice; k < a.r; k += S) {
    const float u = e4m3_to_float(a.U[(int64_t)k * m + rr]);
#pragma unroll
    for (int t = 0; t < B; ++t) acc[t] = fmaf(u, a.y[(int64_t)t * a.r + k], acc[t]);
  }
  // slices of a wave, then the four waves in order
  __syncthreads();
  float* red = row_lds;   // [4][B][R]
#pragma unroll
  for (int t = 0; t < B; ++t) {
#pragma unroll
    for (int mask = R; mask < 64; mask <<= 1) acc[t] += __shfl_xor(acc[t], mask);
    if (lane < R) red[((tid >> 6) * B + t) * R + lane] = acc[t];
  }
  __syncthreads();
  if (tid < B * R) {
    const int t = tid / R, i = tid - t * R;
    const int orow = q * R + i;
    if (orow < m)
      a.O[(int64_t)t * a.ldo + orow] = ((red[t * R + i] + red[(B + t) * R + i]) + red[(2 * B + t) * R + i]) + red[(3 * B + t) * R + i];
  }
}

// ---- many tokens: 16-bit matrix cores -----------------------------------------------------------
// O = X~ Dequant^T as a GEMM on the float16 matrix instruction.  code - zero is an integer of at most eight bits and a
// sign: exact in float16.  X~ comes from float64 as the sum of a float16 and 2^-12 of another, each rounded to nearest, of a
// token's own power of two: it is off by at most 2^-23 of itself, or 2^-47 of the token's largest |x| where that is more (an
// entry 2^23 times the others leaves them theirs).  The second pieces meet codes times 2^-12, which are raised to the codes
// themselves for the first pieces by a multiplication per pair: without it the second bound would be
// 2^-35, and a massive entry that meets a zero weight would cost its row the bits of all others (the tile kernel 3 % faster).  What
// two pieces do not hold, and scales that would leave float32's range in the token's unit, take plain_product.  The products are exact
// in float32 and only its sums round; with two of them per weight fewer do than with the three truncated bfloat16
// pieces that hold a float32 exactly, and the distance from the float64 product is smaller everywhere it was measured
// (512 to 11008 columns, 5 to 4000 tokens, groups of 64 and 128, 2 to 8 bits, 110 sizes: 0.62 to 1.83e-7 of its norm, 0.66 to
// 1.93e-7 with three pieces): the second pieces' products, 2^-11 of the others, go first.  The group's scale is applied to the
// accumulators where a group ends, the token's power of two at the end.
//
// A workgroup takes 32 TT tokens x 128 RT rows of the weight, a wave 32 TT x 32 RT, and walks over chunks of
// 32 columns.  A lane of a wave is row l % 32, and half-wave h = l / 32 takes codes [16 h, 16 h + 16) of the chunk, in the
// order in which they leave their words two at a time (code_order): the contraction index may be dealt out in any order that
// both operands share, and the input's launch writes X~ in that one.  A pair costs an and-or and a packed multiply-add.
// One barrier per chunk, in the middle of its MFMAs; what a chunk needs was requested four chunks before, straight into LDS.
// Between two MFMAs a wave issues a pair or two of the next chunk's codes, a fragment read or a request, in the order
// written down: 2 waves per SIMD, 64 tokens, at most 250 registers.
// Bound: MFMA and what a wave issues beside it (per chunk 16 MFMAs, some 70 other vector and 80 scalar instructions, 12 LDS reads;
// every group, 128 multiply-adds).  Kernel alone, 512 tokens x 4096 x 11008, 3 bits: 100 us (three bfloat16 pieces, split where
// they were staged: 150).
// Whole calls with 16 ranks, 4 bits, three pieces -> now: 512 x 4096 x 11008 166 -> 121 us, 2048 x 11008 x 4096 562 -> 378,
// 4000 x 999 x 1024 71 -> 50, 128 x 4096 x 4096 46 -> 38, 32 x 11008 x 4096 45 -> 29, 8 x 4096 x 4096 21 -> 19.3.
template <int BITS> struct HalfWords { uint32_t w[BITS == 2 ? 1 : (BITS == 8 ? 4 : 2)]; };

// two bfloat16 numbers from floats whose low halves are zero (or are to be dropped)
__device__ __forceinline__ uint32_t pair_high(float a, float b) { return pair_high(__float_as_uint(a), __float_as_uint(b)); }

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

// The order in which a lane's 16 codes of a half chunk leave the words that hold them, two at a time: codes 16 bits apart
// (3 bits: after one shift) need one operation for the pair.  Position p holds code (order >> 4 p) & 15.
template <int BITS>
constexpr uint64_t code_order() {
  uint64_t o = 0;
  for (int q = 0; q < 8; ++q) {
    uint64_t a = 0, b = 0;
    if (BITS == 2) { a = q; b = a + 8; }
    else if (BITS == 3) { a = q < 5 ? q : q + 5; b = q < 5 ? q + 5 : q + 8; }
    else if (BITS == 4) { a = (q & 3) + 8 * (q >> 2); b = a + 4; }
    else { a = 2 * q; b = a + 1; }
    o |= (a | b << 4) << (8 * q);
  }
  return o;
}

template <int BITS>
constexpr uint64_t code_place() {   // the other way round: code j is at position (place >> 4 j) & 15
  uint64_t o = 0;
  for (int p = 0; p < 16; ++p) o |= (uint64_t)p << (4 * (code_order<BITS>() >> (4 * p) & 15));
  return o;
}

// Two codes at bit S of a word's halves, minus the zero, as float16 and in the second pieces' unit: put into the mantissa
// of 1024 (unit 2^-S of it), then one multiply-add; every value on the way is exact.  offset = -(2^(10 - S) + zero) 2^-kSecond.
template <int S, int BITS>
__device__ __forceinline__ f16x2 code_pair(uint32_t w, uint32_t magic, f16x2 offset) {
  constexpr uint32_t one = ((1u << BITS) - 1u) << S, both = one | one << 16;
  const f16x2 v = __builtin_bit_cast(f16x2, (w & both) | magic);
  constexpr _Float16 unit = (_Float16)(1.0f / (1 << (S + kSecond)));
  return __builtin_elementwise_fma(v, f16x2{unit, unit}, offset);
}

// a half chunk's words with codes 16 bits apart
template <int BITS>
__device__ __forceinline__ void align_codes(HalfWords<BITS>& v, int h) {
  if constexpr (BITS == 3) {
    const uint32_t top = v.w[1] >> (16 * h), low = __builtin_amdgcn_alignbit(v.w[1], v.w[0], 16 * h);   // 48 bits
    const uint32_t r = __builtin_amdgcn_alignbit(top, low, 30);
    v.w[0] = (low & 0x7fffu) | ((low << 1) & ~0x7fffu);   // codes 0 .. 4 and, from bit 16, 5 .. 9
    v.w[1] = (r & 0x1ffu) | ((r << 7) & ~0x1ffu);         // codes 10 .. 12 and, from bit 16, 13 .. 15
  }
}

// what a group's zero makes of the offsets of code_pair, for the places that codes take
template <int BITS> struct Offsets { f16x2 o[BITS == 8 ? 1 : (BITS == 4 ? 2 : 3)]; };
template <int BITS>
__device__ __forceinline__ Offsets<BITS> code_offsets(uint32_t zero) {
  constexpr int kStep = BITS == 3 ? 3 : (BITS == 4 ? 4 : 2), kCount = sizeof(Offsets<BITS>) / sizeof(f16x2);
  const _Float16 z1 = (_Float16)(uint16_t)zero;
  const f16x2 z = {z1, z1};
  Offsets<BITS> out;
#pragma unroll
  for (int i = 0; i < kCount; ++i) {
    const _Float16 base = (_Float16)(float)(1 << (10 - kStep * i)), unit = (_Float16)(-1.0f / (1 << kSecond));
    out.o[i] = (f16x2{base, base} + z) * unit;
  }
  return out;
}

// pair q of a half chunk's codes in their order, minus the zero, times 2^-kSecond
template <int BITS, int Q>
__device__ __forceinline__ f16x2 widen_pair(const HalfWords<BITS>& v, uint32_t magic, const Offsets<BITS>& o) {
  if constexpr (BITS == 8) {   // bytes 2 (q % 2) and the next of a word, 0x64 above each
    constexpr _Float16 unit = (_Float16)(1.0f / (1 << kSecond));
    return __builtin_elementwise_fma(
        __builtin_bit_cast(f16x2, __builtin_amdgcn_perm(magic, v.w[Q >> 1], Q & 1 ? 0x05030502u : 0x05010500u)), f16x2{unit, unit}, o.o[0]);
  } else if constexpr (BITS == 4) {
    constexpr int k = Q >> 2, i = Q & 3;
    return code_pair<4 * (i & 1), 4>(i & 2 ? v.w[k] >> 8 : v.w[k], magic, o.o[i & 1]);
  } else if constexpr (BITS == 2) {
    return code_pair<2 * (Q % 3), 2>(v.w[0] >> (6 * (Q / 3)), magic, o.o[Q % 3]);
  } else if constexpr (Q < 5) {
    return code_pair<3 * (Q % 3), 3>(v.w[0] >> (9 * (Q / 3)), magic, o.o[Q % 3]);
  } else {
    return code_pair<3 * (Q - 5), 3>(v.w[1], magic, o.o[Q - 5]);
  }
}

// The three truncated bfloat16 pieces of two floats, paired.  An infinity is its first piece alone, so that its
// products are those of the float32.
__device__ __forceinline__ void split3(float a, float b, uint32_t (&p)[3]) {
  auto rest = [](float v) {
    const float r = v - __uint_as_float(__float_as_uint(v) & 0xffff0000u);
    return __builtin_isinf(v) ? 0.f : r;
  };
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    p[i] = pair_high(a, b);
    a = rest(a);
    b = rest(b);
  }
}

// What a chunk needs goes from memory straight into LDS (buffer_load ... lds), into a ring of kTileRing chunks for each
// half of a workgroup: the tokens' rows of X~, 128 bytes each, [piece][32], whose 16-byte slot k lies at k ^ (token / 2 % 8), so
// that the fragment reads of sixteen neighbouring lanes cover the 64 banks; and, a wave's own 64 rows of the weight at a time,
// the codes' words as they lie in memory, the scales and the zeros (a dword each).  These requests are issued by inline assembly
// and waited for by count: the compiler would wait for all of them before each LDS read.
constexpr int kTileRing = 4;
constexpr int kTileRow = 2 * kChunk * (int)sizeof(uint16_t);
constexpr int kYPitch = 40;   // bfloat16 elements per staged row of 32 ranks

__device__ __forceinline__ int tile_key(int token) { return (token >> 1) & 7; }

__device__ __forceinline__ void buffer_advance(i32x4& b, uint64_t bytes) {
  const uint64_t a = (((uint64_t)(uint32_t)b[1] << 32) | (uint32_t)b[0]) + bytes;
  b[0] = (int)__builtin_amdgcn_readfirstlane((uint32_t)a);
  b[1] = (int)__builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
}

// LDS of one half of a workgroup, in bytes: rows of X~, words, scales, zeros
template <int BITS, int TT>
struct TileLds {
  static constexpr int kX = 32 * TT * kTileRow, kW = 256 * 4 * BITS, kGrid = 256 * 4;   // of one chunk
  static constexpr int w = kTileRing * kX, scale = w + kTileRing * kW, zero = scale + kTileRing * kGrid, all = zero + kTileRing * kGrid;
};

// One token and a row of the weight over chunks [c_begin, c_end), X~ in float32, the sums of eight products in float32 and all
// others in float64: for the few tokens that the pieces do not hold (exponent kPlain), and for rows with scales past kScaleLimit.  The arguments are fetched anew: kept for this, they would fill
// the scalar registers of the loop before it.
template <int BITS>
__device__ __forceinline__ float plain_product(int token, int exponent, int row, int c_begin, int c_end) {
  auto args = (const __attribute__((address_space(4))) ForwardArgs*)__builtin_amdgcn_kernarg_segment_ptr();   // the first argument
  asm volatile("" : "+s"(args));
  const struct { const uint32_t* packed; const float* scales; const uint8_t* zeros; const float* xt; int m, xt_tokens; } a{
      args->packed, args->scales, args->zeros, args->xt, args->m, args->xt_tokens};
  const int gpc = args->group / kChunk;
  // four chunks on their way at a time; lane j (and j + 32) holds x of a chunk's column j
  constexpr int kAhead = 4;
  constexpr uint64_t place = code_place<BITS>();
  const int lane = threadIdx.x & 63, column = lane & 31;
  const int at = (column & 16) + (int)((place >> (4 * (lane & 15))) & 15);
  double total = 0.0, acc = 0.0;
#pragma unroll 1
  for (int c0 = c_begin; c0 < c_end; c0 += kAhead) {
    Words<BITS> words[kAhead];
    float zero[kAhead], scale[kAhead], xv[kAhead];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
      const int c = min(c0 + i, c_end - 1);
      const int64_t grid = (int64_t)(c / gpc) * a.m + row;
      words[i] = *reinterpret_cast<const Words<BITS>*>(a.packed + ((int64_t)c * a.m + row) * BITS);
      zero[i] = (float)a.zeros[grid];
      scale[i] = a.scales[grid];
      const float* x = a.xt + ((int64_t)c * a.xt_tokens + token) * kChunk;
      const _Float16* pieces = reinterpret_cast<const _Float16*>(x) + at;
      xv[i] = exponent == kPlain ? x[column]
                                 : (float)ldexp((double)(float)pieces[0] + (double)(float)pieces[kChunk] * (1.0 / (1 << kSecond)), exponent);
    }
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
      if (c0 + i >= c_end) break;
      static_for<4>([&](auto quarter) {
        constexpr int Q = decltype(quarter)::value;
        float f[8], sum = 0.f;
        codes_to_float<BITS, Q>(words[i], f);
#pragma unroll
        for (int j = 0; j < 8; ++j)
          sum = fmaf(f[j] - zero[i], __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(xv[i]), 8 * Q + j)), sum);
        acc += (double)sum;
      });
      if ((c0 + i + 1) % gpc == 0 || c0 + i + 1 == c_end) {
        total = fma((double)scale[i], acc, total);
        acc = 0.0;
      }
    }
  }
  return (float)total;
}

// Largest and, but for zero, smallest scale whose products with the accumulators stay in float32's normal range before a
// token's power of two is taken off: the accumulators are multiples of 2^-37 below 2^40.
constexpr uint32_t kScaleLimit[2] = {(127 - 80) << 23, (127 + 80) << 23};   // 2^-80, 2^80

struct TilePlan {
  int token_blocks, row_blocks, splits, chunks_per_part;   // splits x KG parts
};

template <int BITS, int TT, int RT, int KG>
__global__ __launch_bounds__(256 * KG, 2) void forward_tile_kernel(ForwardArgs a, int tokens, TilePlan plan) {
  constexpr int kTokens = 32 * TT, kRows = 128 * RT;
  using Lds = TileLds<BITS, TT>;
  extern __shared__ __attribute__((aligned(16))) char tile_lds[];
  typedef __attribute__((address_space(3))) char lds_char;
  const int part = KG == 1 ? 0 : (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
  const int tid = threadIdx.x & 255, lane = tid & 63, wave = (int)__builtin_amdgcn_readfirstlane(tid >> 6), h = lane >> 5;
  const int m = a.m, chunks = a.n / kChunk, gpc = a.group / kChunk;
  // Consecutive items of one XCD (workgroup ids = x mod 8) share a split and neighbouring tiles
  const int total_items = plan.token_blocks * plan.row_blocks * plan.splits;
  const int per = (total_items + 7) / 8;
  const int q = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per || q >= total_items) return;
  const int split = q / (plan.token_blocks * plan.row_blocks);
  const int rem = q - split * plan.token_blocks * plan.row_blocks;
  const int rb = rem / plan.token_blocks, tb = rem - rb * plan.token_blocks;
  const int c_begin = min(chunks, (split * KG + part) * plan.chunks_per_part);
  const int c_end = min(chunks, c_begin + plan.chunks_per_part);

  static_assert(RT == 2, "a wave's rows are 64: a request's lanes");
  uint32_t row[RT];   // within the workgroup's rows; rows past the last one repeat it, not stored
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
    row[rt] = (uint32_t)min((wave * RT + rt) * 32 + (lane & 31), m - 1 - rb * kRows);
  const uint8_t* u_codes = a.U + (int64_t)rb * kRows;

  const int exponent = a.exponents[min(tb * kTokens + lane, tokens - 1)];   // a token's per lane

  // Batch j of requests: X~ of chunk j (counted from c_begin), words and grids of chunk j + 1.  What lies past the part's
  // end is its last chunk again.
  const int count = max(c_end - c_begin, 1);                  // chunks that can be asked for
  const int c_first = min(c_begin, chunks - 1);
  const int row0 = rb * kRows + wave * 64, rows_left = min(max(m - row0, 0), 64);
  const int row_at = min(row0, m - 1);                        // a base inside the arrays
  const uint32_t x_step = (uint32_t)(a.xt_tokens * kTileRow);
  const uint64_t w_step = (uint64_t)m * (4 * BITS);
  const i32x4 x_src = buffer_at(reinterpret_cast<const char*>(a.xt) + (int64_t)tb * kTokens * kTileRow,
                                ((int64_t)chunks * a.xt_tokens - tb * kTokens) * kTileRow);
  i32x4 w_src = buffer_at(a.packed + ((int64_t)c_first * m + row_at) * BITS, rows_left * (4 * BITS));
  i32x4 scale_src = buffer_at(a.scales + (int64_t)(c_first / gpc) * m + row_at, rows_left * 4);
  i32x4 zero_src = buffer_at(a.zeros + (int64_t)(c_first / gpc) * m + row_at, rows_left);
  uint32_t x_at_chunk = (uint32_t)c_first * x_step;
  int x_count = 1, w_count = 1, w_left = gpc - c_first % gpc;
  uint32_t x_off[TT];
#pragma unroll
  for (int i = 0; i < TT; ++i) {   // 8 tokens a request; tokens past the last repeat it, not stored
    const int t = (wave * TT + i) * 8 + (lane >> 3);
    x_off[i] = (uint32_t)(min(t, tokens - 1 - tb * kTokens) * kTileRow + (((lane & 7) ^ tile_key(t)) << 4));
  }
  const uint32_t lane4 = (uint32_t)lane * 4, lane16 = (uint32_t)lane * 16;
  const int part_at = part * Lds::all;
  const uint32_t lbase = (uint32_t)(uintptr_t)(lds_char*)tile_lds + (uint32_t)part_at;
  const uint32_t x_dst = lbase + (uint32_t)(wave * TT * 1024), w_dst = lbase + (uint32_t)(Lds::w + wave * (256 * BITS)),
                 grid_dst = lbase + (uint32_t)(Lds::scale + wave * 256);
  constexpr int kWide = BITS % 4 == 0 ? 16 : 4, kWordRequests = 256 * BITS / (64 * kWide);
  constexpr int kBatch = TT + kWordRequests + 2;
  // A request of a batch, the words last.  words: where they go, relative to the ring
  auto request = [&](auto index, auto slot_x, auto slot_grid, uint32_t words) {
    constexpr int I = decltype(index)::value, S = decltype(slot_grid)::value;
    if constexpr (I < TT) {
      request_to_lds<16>(x_src, x_off[I], x_at_chunk, x_dst + decltype(slot_x)::value * Lds::kX + I * 1024);
    } else if constexpr (I == TT) {
      request_to_lds<4>(scale_src, lane4, 0, grid_dst + S * Lds::kGrid);
    } else if constexpr (I == TT + 1) {
      request_to_lds<1>(zero_src, (uint32_t)lane, 0, grid_dst + (Lds::zero - Lds::scale) + S * Lds::kGrid);
    } else {
      constexpr int k = I - TT - 2;
      request_to_lds<kWide>(w_src, (kWide == 16 ? lane16 : lane4) + k * 64 * kWide, 0, w_dst + words + k * 64 * kWide);
    }
  };
  auto advance_x = [&]() {
    if (x_count < count) x_at_chunk += x_step;
    ++x_count;
  };
  auto advance_w = [&]() {
    const bool more = w_count < count;
    buffer_advance(w_src, more ? w_step : 0);
    const bool next_group = more && --w_left == 0;
    buffer_advance(scale_src, next_group ? 4u * (uint32_t)m : 0u);
    buffer_advance(zero_src, next_group ? (uint32_t)m : 0u);
    if (next_group) w_left = gpc;
    ++w_count;
  };

  // what is read back: fragments of X~ (piece p, step ks: its place in a token's row), words, scales and zeros
  uint32_t x_at[2][2];
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
      x_at[p][ks] = (uint32_t)(part_at + (lane & 31) * kTileRow + (((4 * p + 2 * h + ks) ^ tile_key(lane & 31)) << 4));
  const uint32_t w_at = (uint32_t)(part_at + Lds::w + wave * (256 * BITS) + (lane & 31) * (4 * BITS) + h * (BITS <= 3 ? 4 : 2 * BITS));
  const uint32_t grid_at = (uint32_t)(part_at + Lds::scale + wave * 256 + (lane & 31) * 4);
  auto lds_at = [&](uint32_t at) { return (const lds_char*)tile_lds + at; };
  auto lds_word = [&](uint32_t at) { return *(const __attribute__((address_space(3))) uint32_t*)lds_at(at); };
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  struct Raw { HalfWords<BITS> w[RT]; float scale[RT]; uint32_t zero[RT]; };
  auto read_raw = [&](Raw& r, auto slot_, uint32_t words, auto rt_) {
    constexpr int slot = decltype(slot_)::value, rt = decltype(rt_)::value;
    const uint32_t at = w_at + words + rt * 32 * (4 * BITS);
    if constexpr (BITS == 2) r.w[rt].w[0] = lds_word(at);
    else if constexpr (BITS == 3) { r.w[rt].w[0] = lds_word(at); r.w[rt].w[1] = lds_word(at + 4); }
    else if constexpr (BITS == 4) { const u32x2 q = *(const __attribute__((address_space(3))) u32x2*)lds_at(at); r.w[rt].w[0] = q.x; r.w[rt].w[1] = q.y; }
    else { const u32x4 q = *(const __attribute__((address_space(3))) u32x4*)lds_at(at); r.w[rt].w[0] = q.x; r.w[rt].w[1] = q.y; r.w[rt].w[2] = q.z; r.w[rt].w[3] = q.w; }
    r.scale[rt] = __uint_as_float(lds_word(grid_at + slot * Lds::kGrid + rt * 128));
    r.zero[rt] = lds_word(grid_at + (Lds::zero - Lds::scale) + slot * Lds::kGrid + rt * 128);
  };

  f32x16 acc[TT][RT], total[TT][RT];
#pragma unroll
  for (int tt = 0; tt < TT; ++tt)
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int r = 0; r < 16; ++r) { acc[tt][rt][r] = 0.f; total[tt][rt][r] = 0.f; }

  uint32_t least = ~0u, most = 0;   // scales of the lane's rows: magnitude less one, magnitude
  auto flush = [&](const float (&sc)[RT]) {
#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          total[tt][rt][r] = fmaf(sc[rt], acc[tt][rt][r], total[tt][rt][r]);
          acc[tt][rt][r] = 0.f;
        }
  };

  constexpr int kHalf = 2 * TT * RT;   // MFMAs of one piece
  Raw raw[2];
  f16x8 fr[2][2][TT];    // [piece][16 columns]
  struct Codes { f16x2 pair[RT][8]; float scale[RT]; } codes[2];
  uint32_t magic = 0x64006400u;
  asm volatile("" : "+v"(magic));   // in a vector register, so that mask and 1024 go into one instruction
  Offsets<BITS> off[RT];
  auto start_codes = [&](Raw& r, Codes& to) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      off[rt] = code_offsets<BITS>(r.zero[rt]);
      align_codes<BITS>(r.w[rt], h);
      to.scale[rt] = r.scale[rt];
    }
  };
  auto kept = [](f16x2 v) {   // formed here, not where a later step uses it
    uint32_t bits = __builtin_bit_cast(uint32_t, v);
    asm volatile("" : "+v"(bits));
    return __builtin_bit_cast(f16x2, bits);
  };
  auto widen = [&](Raw& r, Codes& to, auto index) {   // pair by pair, index < 8 RT
    constexpr int I = decltype(index)::value, q = I / RT, rt = I % RT;
    to.pair[rt][q] = kept(widen_pair<BITS, q>(r.w[rt], magic, off[rt]));
  };
  auto raise = [&](Codes& to, auto step_, auto index) {   // from the second pieces' unit to the first's: four pairs of a step, index < 4 RT
    constexpr int q = 4 * decltype(step_)::value + decltype(index)::value / RT, rt = decltype(index)::value % RT;
    constexpr _Float16 unit = (_Float16)(float)(1 << kSecond);
    to.pair[rt][q] = kept(to.pair[rt][q] * f16x2{unit, unit});
  };
  auto read_x = [&](auto slot_, auto piece, auto index) {   // index < 2 TT
    constexpr int p = decltype(piece)::value, ks = decltype(index)::value / TT, tt = decltype(index)::value % TT;
    fr[p][ks][tt] = *(const __attribute__((address_space(3))) f16x8*)lds_at(x_at[p][ks] + decltype(slot_)::value * Lds::kX + tt * 32 * kTileRow);
  };
  auto mfma = [&](const Codes& b, auto piece, auto index) {   // index < kHalf
    constexpr int I = decltype(index)::value, p = decltype(piece)::value;
    constexpr int ks = I / (TT * RT), tt = I / RT % TT, rt = I % RT;
    struct Quad { f16x2 e[4]; };
    const f16x8 bv = __builtin_bit_cast(f16x8, Quad{{b.pair[rt][4 * ks], b.pair[rt][4 * ks + 1], b.pair[rt][4 * ks + 2], b.pair[rt][4 * ks + 3]}});
    acc[tt][rt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fr[p][ks][tt], bv, acc[tt][rt], 0, 0, 0);
  };
  using std::integral_constant;
  typedef integral_constant<int, 0> Zero;
  typedef integral_constant<int, 1> One;

  // chunk 0's words and grids, batches 0 and 1; when those words are read, batches 2 and 3
  auto batch = [&](auto index, auto from) {
    constexpr int J = decltype(index)::value, F = decltype(from)::value;
    static_for<kBatch - F>([&](auto k) {
      request(integral_constant<int, F + decltype(k)::value>{}, integral_constant<int, (J < 0 ? 0 : J)>{},
              integral_constant<int, (J + 1) % kTileRing>{}, (J + 1) % kTileRing * Lds::kW);
    });
    if constexpr (J >= 0) advance_x();
    advance_w();
  };
  batch(integral_constant<int, -1>{}, integral_constant<int, TT>{});
  batch(Zero{}, Zero{});
  batch(One{}, Zero{});
  wait_requests<kBatch>();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  static_for<RT>([&](auto rt) { read_raw(raw[0], Zero{}, 0u, rt); });
  static_for<RT>([&](auto rt) { read_raw(raw[1], One{}, (uint32_t)Lds::kW, rt); });
  static_for<2 * TT>([&](auto k) { read_x(Zero{}, One{}, k); });
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  batch(integral_constant<int, 2>{}, Zero{});
  batch(integral_constant<int, 3>{}, Zero{});
  start_codes(raw[0], codes[0]);
  static_for<8 * RT>([&](auto k) { widen(raw[0], codes[0], k); });

  // Step j: the MFMAs of chunk j's second pieces (the smaller ones first) | barrier | those of the first.  At the barrier every wave has read
  // all it needs of chunk j's rows and of chunk j + 1's words, whose places batch j + 4 takes, and batch j + 1 has
  // landed: the newest requests are those of batches j + 2 and j + 3.  Beside the MFMAs, chunk j + 1's codes are widened and
  // what comes next is read from LDS, in the order written down here (a step is one basic block; left to the
  // scheduler, the MFMAs follow each other and the vector instructions follow them).
  int left = gpc - c_begin % gpc;   // chunks until the group ends
  auto step = [&](auto slot_, int c) {
    constexpr int Q = decltype(slot_)::value, P = Q & 1;
    typedef integral_constant<int, Q> Here;
    typedef integral_constant<int, (Q + 1) % kTileRing> Next;
    typedef integral_constant<int, (Q + 2) % kTileRing> After;
    constexpr int kPairs = 8 * RT / (2 * kHalf);   // widened per MFMA
    constexpr int kRaised = 8 * RT / kHalf;        // raised per MFMA: a step's pairs while the other step's MFMAs go
    start_codes(raw[P ^ 1], codes[P ^ 1]);
    static_for<kHalf>([&](auto i_) {
      constexpr int i = decltype(i_)::value;
      mfma(codes[P], One{}, i_);
      if constexpr (i < 2 * TT) read_x(Here{}, Zero{}, i_);
      static_for<kPairs>([&](auto k) { widen(raw[P ^ 1], codes[P ^ 1], integral_constant<int, kPairs * i + decltype(k)::value>{}); });
      if constexpr (i >= kHalf / 2)
        static_for<kRaised>([&](auto k) { raise(codes[P], Zero{}, integral_constant<int, kRaised * (i - kHalf / 2) + decltype(k)::value>{}); });
      __builtin_amdgcn_sched_barrier(0);
    });
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    wait_requests<(kTileRing - 2) * kBatch>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    static_for<kHalf>([&](auto i_) {
      constexpr int i = decltype(i_)::value;
      mfma(codes[P], Zero{}, i_);
      if constexpr (i >= kHalf / 2) read_x(Next{}, One{}, integral_constant<int, i - kHalf / 2>{});   // kHalf / 2 = 2 TT
      if constexpr (i < RT) read_raw(raw[P], After{}, After::value * Lds::kW, i_);
      static_for<kPairs>([&](auto k) { widen(raw[P ^ 1], codes[P ^ 1], integral_constant<int, kPairs * (kHalf + i) + decltype(k)::value>{}); });
      if constexpr (i < kHalf / 2)
        static_for<kRaised>([&](auto k) { raise(codes[P], One{}, integral_constant<int, kRaised * i + decltype(k)::value>{}); });
      static_for<(kBatch + kHalf - 1) / kHalf>([&](auto k) {
        constexpr int r = i * ((kBatch + kHalf - 1) / kHalf) + decltype(k)::value;
        if constexpr (r < kBatch) request(integral_constant<int, r>{}, Here{}, Next{}, Next::value * Lds::kW);
      });
      __builtin_amdgcn_sched_barrier(0);
    });
    advance_x();
    advance_w();
    if (c < c_end && (--left == 0 || c + 1 == c_end)) {   // the same for a wave
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const uint32_t v = __float_as_uint(codes[P].scale[rt]) & 0x7fffffffu;
        least = min(least, v - 1);
        most = max(most, v);
      }
      flush(codes[P].scale);
      left = gpc;
    }
  };
  // the same count for all waves; past c_end a part adds what is never used
  int c = c_begin;
  const int stop = c_begin + plan.chunks_per_part;
  for (; c + kTileRing <= stop; c += kTileRing) {
    step(integral_constant<int, 0>{}, c);
    step(integral_constant<int, 1>{}, c + 1);
    step(integral_constant<int, 2>{}, c + 2);
    step(integral_constant<int, 3>{}, c + 3);
  }
  if (c < stop) {
    step(integral_constant<int, 0>{}, c);
    if (c + 1 < stop) {
      step(integral_constant<int, 1>{}, c + 1);
      if (c + 2 < stop) step(integral_constant<int, 2>{}, c + 2);
    }
  }
  wait_requests<0>();
  __syncthreads();   // the ring's space is used for other things from here on

  // back from the pieces' unit: accumulator r of a lane is token (r / 4) * 8 + (lane / 32) * 4 + r % 4 of its tile
#pragma unroll
  for (int tt = 0; tt < TT; ++tt)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int e = __shfl(exponent, tt * 32 + (r >> 2) * 8 + h * 4 + (r & 3));
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) total[tt][rt][r] = ldexpf(total[tt][rt][r], e);
    }

  // tokens whose X~ is not in pieces; all, if a scale is too large or too small
  const int there = min(kTokens, tokens - tb * kTokens);
  const bool extreme = least < kScaleLimit[0] - 1 || most > kScaleLimit[1];
  const uint64_t plain = (__ballot(extreme) ? ~0ull : __ballot(exponent == kPlain)) & (~0ull >> (64 - there));
#pragma unroll 1
  for (uint64_t rest = plain; rest; rest &= rest - 1) {
    const int t = __builtin_ctzll(rest);
    const float sum = plain_product<BITS>(tb * kTokens + t, __builtin_amdgcn_readlane(exponent, t), min(row0 + lane, m - 1), c_begin, c_end);   // a row per lane
    float mine[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) mine[rt] = __shfl(sum, rt * 32 + (lane & 31));
#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const bool here = t == tt * 32 + (r >> 2) * 8 + h * 4 + (r & 3);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) total[tt][rt][r] = here ? mine[rt] : total[tt][rt][r];
      }
  }

  // The low-rank part, once: coefficients y (tokens x r) against the e4m3 codes of U, 32 ranks at a time; e4m3
  // is exact in bfloat16, y goes through three pieces of it (exact in float32, and their range is its range).
  if (a.r > 0 && split == plan.splits - 1) {
    constexpr int E = TT == 1 ? 4 : 8;   // consecutive ranks a thread stages: 256 E = 32 kTokens
#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[tt][rt][r] = 0.f;
    auto ys = reinterpret_cast<uint16_t(*)[kTokens][kYPitch]>(tile_lds) + 3 * part;
    const int y_tok = tid / (32 / E), y_col = (tid % (32 / E)) * E;
    const int64_t y_row = (int64_t)min(tb * kTokens + y_tok, tokens - 1) * a.r;
#pragma unroll 1
    for (int k0 = 32 * part; k0 < a.r + 32 * part; k0 += 32 * KG) {   // the same count for all waves
      float yv[E];
#pragma unroll
      for (int i = 0; i < E; ++i) {
        const int k = min(k0 + y_col + i, a.r - 1);
        float v;
        if (a.y_parts) {
          double part[kCoeffSplits], sum = 0.0;
#pragma unroll
          for (int q = 0; q < kCoeffSplits; ++q)   // issued whatever the split: no wait between them
            part[q] = a.y_parts[(int64_t)min(q, a.y_splits - 1) * tokens * a.r + y_row + k];
#pragma unroll
          for (int q = 0; q < kCoeffSplits; ++q) sum += q < a.y_splits ? part[q] : 0.0;
          v = (float)(sum * (double)fp16_bits_to_float(a.sigma[k]));
        } else {
          v = a.y[y_row + k];
        }
        yv[i] = k0 + y_col + i < a.r ? v : 0.f;
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < E; i += 4) {
        uint32_t lo[3], hi[3];   // a coefficient past the float32 range makes its products infinite
        split3(yv[i], yv[i + 1], lo);
        split3(yv[i + 2], yv[i + 3], hi);
#pragma unroll
        for (int k = 0; k < 3; ++k) *reinterpret_cast<uint2*>(&ys[k][y_tok][y_col + i]) = make_uint2(lo[k], hi[k]);
      }
      bf16x8 u[2][RT];
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          float f[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const int k = k0 + 16 * h + 8 * ks + j;
            const float v = e4m3_to_float(u_codes[(int64_t)min(k, a.r - 1) * m + row[rt]]);
            f[j] = k < a.r ? v : 0.f;
          }
          const uint4 o = make_uint4(pair_high(f[0], f[1]), pair_high(f[2], f[3]), pair_high(f[4], f[5]), pair_high(f[6], f[7]));
          u[ks][rt] = __builtin_bit_cast(bf16x8, o);
        }
      __syncthreads();
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int p = 2; p >= 0; --p)   // the smallest piece first
#pragma unroll
          for (int tt = 0; tt < TT; ++tt) {
            const bf16x8 av = *reinterpret_cast<const bf16x8*>(&ys[p][tt * 32 + (lane & 31)][16 * h + 8 * ks]);
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
              acc[tt][rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, u[ks][rt], acc[tt][rt], 0, 0, 0);
          }
    }
    const float one[RT] = {1.f, 1.f};
    flush(one);
  }

  if constexpr (KG > 1) {   // the second part's sums go to the first through LDS, a tile at a time
    static_assert(KG == 2, "");
    float* ex = reinterpret_cast<float*>(tile_lds) + tid;
#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        __syncthreads();
        if (part == 1) {
#pragma unroll
          for (int r = 0; r < 16; ++r) ex[r * 256] = total[tt][rt][r];
        }
        __syncthreads();
        if (part == 0) {
#pragma unroll
          for (int r = 0; r < 16; ++r) total[tt][rt][r] += ex[r * 256];
        }
      }
    if (part != 0) return;
  }

  const bool direct = split == 0;
  float* out = direct ? a.O : a.partial + (int64_t)(split - 1) * tokens * m;
  const int64_t ld = direct ? a.ldo : m;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int orow = rb * kRows + (wave * RT + rt) * 32 + (lane & 31);
    if (orow >= m) continue;
#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int t = tb * kTokens + tt * 32 + (r >> 2) * 8 + h * 4 + (r & 3);
        if (t < tokens) out[(int64_t)t * ld + orow] = total[tt][rt][r];
      }
  }
}

// O[t][row] = sum over the column splits, in order: the first is in O, the last holds the low-rank part
__global__ __launch_bounds__(256) void forward_tile_finish_kernel(ForwardArgs a, int tokens, int splits) {
  const int row = blockIdx.x * 256 + threadIdx.x;
  const int t0 = blockIdx.y * 4;
  if (row >= a.m) return;
  float out[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) out[t] = a.O[(int64_t)min(t0 + t, tokens - 1) * a.ldo + row];
  const int more = splits - 1;
  for (int sp0 = 0; sp0 < more; sp0 += 8) {
    float v[8][4];
#pragma unroll
    for (int k = 0; k < 8; ++k)
#pragma unroll
      for (int t = 0; t < 4; ++t)   // issued whatever the split: no branch, no wait
        v[k][t] = a.partial[((int64_t)min(sp0 + k, more - 1) * tokens + min(t0 + t, tokens - 1)) * a.m + row];
#pragma unroll
    for (int k = 0; k < 8; ++k)
#pragma unroll
      for (int t = 0; t < 4; ++t) out[t] += sp0 + k < more ? v[k][t] : 0.f;
  }
#pragma unroll
  for (int t = 0; t < 4; ++t)
    if (t0 + t < tokens) a.O[(int64_t)(t0 + t) * a.ldo + row] = out[t];
}

constexpr int kFwdRun = 8;            // chunks: the least a column split keeps
constexpr int kPartialTokens = 32;   // the workspace holds partial sums of 32 tokens for every run of 256 columns

template <int BITS, int TT, int KG>
ptq_status launch_forward_tile_as(const ForwardArgs& a, int tokens, TilePlan p, hipStream_t st) {
  const int chunks = a.n / kChunk;
  p.chunks_per_part = (int)ceil_div(chunks, p.splits * KG);
  p.splits = (int)ceil_div(chunks, (int64_t)p.chunks_per_part * KG);
  const unsigned grid = 8u * (unsigned)ceil_div((int64_t)p.token_blocks * p.row_blocks * p.splits, 8);
  constexpr int ring = KG * TileLds<BITS, TT>::all, ys = KG * 3 * 32 * TT * kYPitch * (int)sizeof(uint16_t);
  constexpr int lds = std::max(std::max(ring, ys), KG > 1 ? 256 * 16 * (int)sizeof(float) : 0);
  if (!lds_opt_in<forward_tile_kernel<BITS, TT, 2, KG>>(lds)) return PTQ_ERR_HIP;
  forward_tile_kernel<BITS, TT, 2, KG><<<grid, 256 * KG, lds, st>>>(a, tokens, p);
  if (p.splits > 1) {
    dim3 gf((unsigned)ceil_div(a.m, 256), (unsigned)ceil_div(tokens, 4));
    forward_tile_finish_kernel<<<gf, 256, 0, st>>>(a, tokens, p.splits);
  }
  return PTQ_OK;
}

template <int BITS>
ptq_status launch_forward_tile(const ForwardArgs& a, int tokens, hipStream_t st) {
  const int chunks = a.n / kChunk;
  const int TT = tokens <= 32 ? 1 : 2;
  TilePlan p{};
  p.token_blocks = (int)ceil_div(tokens, 32 * TT);
  p.row_blocks = (int)ceil_div(a.m, 256);
  const int64_t tiles = (int64_t)p.token_blocks * p.row_blocks;
  // Two waves per SIMD hide each other's waits: where the tiles alone give every compute unit two workgroups the columns
  // stay whole; otherwise a workgroup's two halves take half of its columns each (64 tokens a tile: 512 x 4096 x 11008, 4 bits, 162
  // us and 177 without, with the bfloat16 pieces), and the columns are split over workgroups until every compute unit has
  // one, as far as the partial sums fit the workspace and a part keeps eight chunks.  Up to 32 tokens the codes' stream is
  // the bound and twice as many workgroups, without halves, keep more of it in flight (whole call, 16 ranks: 32 x 11008 x 4096
  // 27.5 us, 31.6 with halves; 8 x 4096 x 4096 18.7 and 19.5; 5 x 777 x 512 16.1 and 16.8).
  const bool many = tiles >= 512;
  int64_t s = many ? 1 : ceil_div(TT == 1 ? 512 : 256, tiles);
  s = std::min<int64_t>(s, ceil_div(chunks, kFwdRun) * kPartialTokens / tokens);
  s = std::max<int64_t>(1, std::min<int64_t>(s, chunks / kFwdRun));
  p.splits = (int)s;
  if (TT == 1) return launch_forward_tile_as<BITS, 1, 1>(a, tokens, p, st);
  const bool halves = !many && chunks / s >= 2;
  return halves ? launch_forward_tile_as<BITS, 2, 2>(a, tokens, p, st) : launch_forward_tile_as<BITS, 2, 1>(a, tokens, p, st);
}

template <int BITS, int B, int R>
ptq_status launch_forward_rows_as(const ForwardArgs& a, hipStream_t st) {
  const int columns = std::min(a.n, kRowLdsFloats / B / kChunk * kChunk);
  const int items = (int)ceil_div(a.m, R);
  const size_t lds = std::max((size_t)B * (columns + columns / kChunk), (size_t)4 * B * R) * sizeof(float);
  if (!lds_opt_in<forward_rows_kernel<BITS, B, R>>(160 * 1024)) return PTQ_ERR_HIP;
  forward_rows_kernel<BITS, B, R><<<8u * (unsigned)ceil_div(items, 8), 256, lds, st>>>(a, columns, items);
  return PTQ_OK;
}

template <int BITS, int B>
ptq_status launch_forward_rows(const ForwardArgs& a, hipStream_t st) {
  return a.m > 2048 ? launch_forward_rows_as<BITS, B, 16>(a, st) : launch_forward_rows_as<BITS, B, 8>(a, st);
}

// One token always, up to four while X~ has at most 16384 values go row by row (whole call, 4 bits, 16 ranks, rows and
// tiles: 2 x 4096 x 4096 14.2 and 18.1 us, 2 x 11008 x 11008 69 and 37, 3 x 11008 x 4096 20.5 and 22.7, 3 x 4096 x 8192 30 and 23,
// 4 x 11008 x 2048 15.5 and 19.1; on the line 2 x 4096 x 8192 22.1 and 22.9, 4 x 4096 x 4096 19.3 and 17.9).
bool takes_tiles(int64_t tokens, int64_t n) { return tokens > 1 && (tokens > 4 || tokens * n > 16384); }

template <int BITS>
ptq_status launch_forward(const ForwardArgs& a, int tokens, hipStream_t st) {
  if (takes_tiles(tokens, a.n)) return launch_forward_tile<BITS>(a, tokens, st);
  switch (tokens) {
    case 1: return launch_forward_rows<BITS, 1>(a, st);
    case 2: return launch_forward_rows<BITS, 2>(a, st);
    case 3: return launch_forward_rows<BITS, 3>(a, st);
    default: return launch_forward_rows<BITS, 4>(a, st);
  }
}

}  // namespace

ptq_status pack_codes_launch(const uint8_t* codes, int64_t ldc, int64_t m, int64_t n, int bits, uint32_t* packed,
                             const float* scales, const uint8_t* zeros, int64_t ng, float* scales_t, uint8_t* zeros_t,
                             hipStream_t st) {
  const int64_t row_tiles = ceil_div(m, 32), tiles = scales ? row_tiles * ceil_div(ng, 32) : 0;
  const GridTranspose t{scales, zeros, (int)ng, scales_t, zeros_t, (int)row_tiles, (int)tiles};
  const unsigned grid = (unsigned)(ceil_div(m * (n / kChunk), 256) + tiles);
  switch (bits) {
    case 2: pack_kernel<2><<<grid, 256, 0, st>>>(codes, ldc, (int)m, (int)n, packed, t); break;
    case 3: pack_kernel<3><<<grid, 256, 0, st>>>(codes, ldc, (int)m, (int)n, packed, t); break;
    case 4: pack_kernel<4><<<grid, 256, 0, st>>>(codes, ldc, (int)m, (int)n, packed, t); break;
    case 8: pack_kernel<8><<<grid, 256, 0, st>>>(codes, ldc, (int)m, (int)n, packed, t); break;
    default: return PTQ_ERR_ARG;
  }
  PTQ_HIP_CHECK_LAUNCH();
  return PTQ_OK;
}

ptq_status unpack_dequant_launch(const uint32_t* packed, int64_t m, int64_t n, int bits, const float* scales,
                                 const uint8_t* zeros, int group, double* Wq, int64_t ldq, hipStream_t st) {
  const unsigned grid = (unsigned)ceil_div(m * (n / kChunk), 256);
  switch (bits) {
    case 2: unpack_dequant_kernel<2><<<grid, 256, 0, st>>>(packed, (int)m, (int)n, scales, zeros, group, Wq, ldq); break;
    case 3: unpack_dequant_kernel<3><<<grid, 256, 0, st>>>(packed, (int)m, (int)n, scales, zeros, group, Wq, ldq); break;
    case 4: unpack_dequant_kernel<4><<<grid, 256, 0, st>>>(packed, (int)m, (int)n, scales, zeros, group, Wq, ldq); break;
    case 8: unpack_dequant_kernel<8><<<grid, 256, 0, st>>>(packed, (int)m, (int)n, scales, zeros, group, Wq, ldq); break;
    default: return PTQ_ERR_ARG;
  }
  PTQ_HIP_CHECK_LAUNCH();
  return PTQ_OK;
}

static size_t forward_partial_bytes(int64_t m, int64_t n) {
  return align_up((size_t)ceil_div(n / kChunk, kFwdRun) * kPartialTokens * (size_t)m * sizeof(float), 256);
}

static size_t forward_tail_bytes(int64_t m) { return align_up((size_t)ceil_div(m, 256) * sizeof(unsigned), 256); }

// ---- scratch for callers that cannot allocate -----------------------------------------------
// One array per GPU, part of the library's code object: the device memory the forward call needs
// beyond its inputs and outputs (the rotated input, the low-rank coefficients, the partial sums of
// the column splits).  Its name is a host-side stand-in, not a device
// address: the address on the current device comes from hipGetSymbolAddress, once per device.
constexpr size_t kStaticScratchBytes = (size_t)32 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

size_t linear_forward_static_scratch_bytes() { return kStaticScratchBytes; }

ptq_status linear_forward_static_scratch(void** ptr) {
  constexpr int kMaxDevices = 64;
  static std::atomic<void*> per_device[kMaxDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return PTQ_ERR_HIP;
  void* p = per_device[dev].load(std::memory_order_acquire);
  if (!p) {
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return PTQ_ERR_HIP;
    per_device[dev].store(p, std::memory_order_release);   // every thread gets the same address: no race
  }
  *ptr = p;
  return PTQ_OK;
}

size_t linear_forward_workspace_bytes(int64_t tokens, int64_t m, int64_t n, int64_t r) {
  return align_up((size_t)tokens * n * sizeof(float), 256) +
         align_up((size_t)tokens * (r > 0 ? r : 1) * sizeof(float), 256) + forward_partial_bytes(m, n) +
         forward_tail_bytes(m);   // which sizes fit the static array is part of the contract
}

ptq_status linear_forward_launch(const void* X, ptq_dtype xdt, int64_t ldx, int64_t tokens, int64_t m, int64_t n,
                                 const uint32_t* packed, int bits, const float* scales, const uint8_t* zeros,
                                 int group, const int32_t* perm, int b_I, int b_H, const uint8_t* U,
                                 const uint8_t* V, const uint16_t* sigma, int r, const double* s, float* O,
                                 int64_t ldo, void* ws, hipStream_t st) {
  char* base = static_cast<char*>(ws);
  float* xt = reinterpret_cast<float*>(base);
  float* y = reinterpret_cast<float*>(reinterpret_cast<char*>(xt) + align_up((size_t)tokens * n * sizeof(float), 256));
  float* partial = reinterpret_cast<float*>(reinterpret_cast<char*>(y) +
                                            align_up((size_t)tokens * (r > 0 ? r : 1) * sizeof(float), 256));
  // behind the partial sums, which leave a split's room: the tokens' exponents, where X~ is in pieces.  A layer of
  // a few rows and more tokens than its workspace has exponents for goes by runs of tokens, each with its exponents at
  // the very end: the last run may be short enough to split its columns.
  const size_t behind = forward_partial_bytes(m, n) + forward_tail_bytes(m);
  const bool pieces = takes_tiles(tokens, n);
  const int64_t run = pieces ? std::min<int64_t>(tokens, (int64_t)(behind / sizeof(int))) : tokens;
  for (int64_t t0 = 0; t0 < tokens; t0 += run) {
    const int part = (int)std::min(run, tokens - t0);
    int* exponents = pieces ? reinterpret_cast<int*>(reinterpret_cast<char*>(partial) + behind) - part : nullptr;
    const char* x0 = static_cast<const char*>(X) + t0 * ldx * (xdt == PTQ_F64 ? 8 : (xdt == PTQ_F32 ? 4 : 2));
    const bool tiles = pieces && takes_tiles(part, n);
    PrepArgs prep{x0, ldx, part, (int)n, perm, b_I, V, sigma, s, r, xt, y, nullptr, 0, 1, 0, 1, 1, 0, exponents, false, 0, 1.0 / std::sqrt((double)b_H)};
    while (1 << prep.lg < b_H) ++prep.lg;
    // the coefficients of many tokens, where the room that the partial sums leave (a split's) holds them: by several workgroups
    if (tiles && r > 0 && part >= kPrepMany) {
      const int64_t wanted = std::min<int64_t>(std::min<int64_t>(n / 1024, kCoeffSplits), 128 / (ceil_div(part, 16) * ceil_div(r, 16)));
      const int64_t held = ceil_div(n / kChunk, kFwdRun) * kPartialTokens;   // tokens times splits
      const int64_t free = (int64_t)behind - std::max<int64_t>(held / part - 1, 0) * part * m * 4;
      const int64_t room = part == tokens ? (free - part * 4 - 8) / (part * r * 8) : 0;
      prep.coeff_splits = (int)std::max<int64_t>(1, std::min(wanted, room));
      if (prep.coeff_splits > 1)
        prep.y_parts = reinterpret_cast<double*>((reinterpret_cast<uintptr_t>(exponents) & ~(uintptr_t)7)) - (int64_t)prep.coeff_splits * part * r;
    }
    if (tiles) prep.order = bits == 2 ? code_order<2>() : (bits == 3 ? code_order<3>() : (bits == 4 ? code_order<4>() : code_order<8>()));
    ptq_status rc;
    switch (xdt) {
      case PTQ_F32: rc = launch_forward_prep<PTQ_F32>(prep, st); break;
      case PTQ_BF16: rc = launch_forward_prep<PTQ_BF16>(prep, st); break;
      case PTQ_F64: rc = launch_forward_prep<PTQ_F64>(prep, st); break;
      default: return PTQ_ERR_DTYPE;
    }
    if (rc != PTQ_OK) return rc;
    ForwardArgs a{packed, scales, zeros, (int)m, (int)n, group, xt, part, y, prep.y_parts, prep.coeff_splits, sigma, U, r, exponents, partial, O + t0 * ldo, ldo};
    switch (bits) {
      case 2: rc = launch_forward<2>(a, part, st); break;
      case 3: rc = launch_forward<3>(a, part, st); break;
      case 4: rc = launch_forward<4>(a, part, st); break;
      case 8: rc = launch_forward<8>(a, part, st); break;
      default: return PTQ_ERR_ARG;
    }
    if (rc != PTQ_OK) return rc;
  }
  PTQ_HIP_CHECK_LAUNCH();
  return PTQ_OK;
}

}  // namespace ptq
