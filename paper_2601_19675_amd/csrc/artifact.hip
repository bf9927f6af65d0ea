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
// codes' stream from memory), more of them in tiles on the bfloat16 matrix cores.
#include <algorithm>
#include <type_traits>

#include "common.h"
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
// X~ = X P Q in float64, written as float32 (xt[chunk][token][32]), and, in float64,
//   y[t][k] = sigma_k * sum_j V[k][j] x[t][j] / s[j].
// The first workgroups take TG tokens x RG ranks of y (1 x 4 while there are few tokens, for the latency; 2 x 16
// from kPrepMany on, where one conversion of V and one quotient x / s then serve several products): 2048 columns at a time,
// four per lane, all loads of a step on their way together; the sums over the 64 lanes are folded by halves, one
// exchange per value pair and step.  The others rotate: a workgroup stages a token's row in LDS and transforms
// `segment` of its 256-column chunks (a row goes to several workgroups while there are few tokens).
// For a token or a few both parts are chains of latencies: one token, 4096 x 4096, 16 ranks 3.8 us for the launch, 7.3 +
// 7.2 as two (a workgroup per row; a workgroup per token and rank).  512 tokens x 4096 x 11008 29.5 us, 29.9 + 132 as
// two (the coefficients mostly divisions and conversions, one of each for every product).  The
// coefficients on the float64 matrix instruction were slower: 16 x 16 tiles of tokens x ranks leave most of
// the chip idle (194 us; a single token 28).
struct PrepArgs {
  const void* X;
  int64_t ldx;
  int tokens, n;
  const int32_t* perm;
  int b_I, b_H;
  const uint8_t* V;
  const uint16_t* sigma;
  const double* s;
  int r;
  float* xt;
  float* y;
  int coeff_tiles, segments, segment;   // chunks per segment
};

constexpr int kPrepThreads = 512, kPrepWaves = kPrepThreads / 64;
constexpr int kPrepMany = 32;   // tokens

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

template <int DT, bool ALIGNED>
__global__ __launch_bounds__(kPrepThreads, 4) void forward_prep_kernel(PrepArgs a) {
  extern __shared__ __attribute__((aligned(16))) char prep_lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if ((int)blockIdx.x < a.coeff_tiles) {
    if (a.tokens >= kPrepMany) low_rank_coefficients<DT, ALIGNED, 2, 16>(a, reinterpret_cast<double*>(prep_lds));
    else low_rank_coefficients<DT, ALIGNED, 1, 4>(a, reinterpret_cast<double*>(prep_lds));
    return;
  }
  const int item = blockIdx.x - a.coeff_tiles;
  const int token = item / a.segments, seg = item - token * a.segments;
  using ST = typename StoredType<DT>::type;
  const ST* src = static_cast<const ST*>(a.X) + (int64_t)token * a.ldx;
  ST* buf = reinterpret_cast<ST*>(prep_lds);
  if constexpr (ALIGNED) {   // n is a multiple of 32
    constexpr int kPer = 16 / (int)sizeof(ST);
    for (int c = tid * kPer; c < a.n; c += kPrepThreads * kPer)
      *reinterpret_cast<uint4*>(buf + c) = *reinterpret_cast<const uint4*>(src + c);
  } else {
    for (int c = tid; c < a.n; c += kPrepThreads) buf[c] = src[c];
  }
  const int nchunk_id = (a.b_I + 255) / 256;                   // chunks of the identity part
  const int nchunk = nchunk_id + (a.n - a.b_I + 255) / 256;    // ... plus those of the rotated part
  const int lg = ilog2(a.b_H);
  const double scale = 1.0 / sqrt((double)a.b_H);
  const int k_end = min(nchunk, (seg + 1) * a.segment);
  __syncthreads();
  for (int k = seg * a.segment + wave; k < k_end; k += kPrepWaves) {
    const bool ident = k < nchunk_id;
    const int cs = ident ? 256 * k : a.b_I + 256 * (k - nchunk_id);
    const int ce = ident ? a.b_I : a.n;
    const int c = cs + 4 * lane;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    if (c < ce) {
      const int4 p = *reinterpret_cast<const int4*>(a.perm + c);
      v[0] = stored_to_f64<DT>(buf[p.x]);
      v[1] = stored_to_f64<DT>(buf[p.y]);
      v[2] = stored_to_f64<DT>(buf[p.z]);
      v[3] = stored_to_f64<DT>(buf[p.w]);
    }
    if (!ident) {
      fwht_chunk(v, lg, lane);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] *= scale;
    }
    if (c < ce)   // c is a multiple of 4
      *reinterpret_cast<float4*>(a.xt + ((int64_t)(c >> 5) * a.tokens + token) * kChunk + (c & 31)) =
          make_float4((float)v[0], (float)v[1], (float)v[2], (float)v[3]);
  }
}

template <int DT>
ptq_status launch_forward_prep(PrepArgs a, hipStream_t st) {
  using ST = typename StoredType<DT>::type;
  const size_t row = (size_t)a.n * sizeof(ST);
  if (row > 160 * 1024) return PTQ_ERR_SHAPE;
  const int nchunk = (a.b_I + 255) / 256 + (a.n - a.b_I + 255) / 256;
  a.coeff_tiles = (int)(a.tokens >= kPrepMany ? ceil_div(a.tokens, 2) * ceil_div(a.r, 16) : a.tokens * ceil_div(a.r, 4));
  // every workgroup of a token stages its whole row: split it only as far as that fills the chip
  a.segments = (int)std::min<int64_t>(ceil_div(nchunk, kPrepWaves), ceil_div(256, a.tokens));
  a.segment = (int)ceil_div(nchunk, a.segments);
  const auto off = [](const void* p) { return reinterpret_cast<uintptr_t>(p) % 16; };
  const bool aligned = off(a.X) == 0 && (a.ldx * sizeof(ST)) % 16 == 0 && (a.r == 0 || (off(a.V) % 4 == 0 && off(a.s) == 0));
  const size_t lds = std::max(row, (size_t)kPrepWaves * 32 * sizeof(double));
  const unsigned grid = (unsigned)(a.coeff_tiles + (int64_t)a.tokens * a.segments);
  if (aligned) {
    if (!lds_opt_in<forward_prep_kernel<DT, true>>(160 * 1024)) return PTQ_ERR_HIP;
    forward_prep_kernel<DT, true><<<grid, kPrepThreads, lds, st>>>(a);
  } else {
    if (!lds_opt_in<forward_prep_kernel<DT, false>>(160 * 1024)) return PTQ_ERR_HIP;
    forward_prep_kernel<DT, false><<<grid, kPrepThreads, lds, st>>>(a);
  }
  return PTQ_OK;
}

struct ForwardArgs {
  const uint32_t* packed;   // (n / 32) x m x BITS words
  const float* scales;      // n / group x m
  const uint8_t* zeros;     // n / group x m
  int m, n, group;
  const float* xt;          // X~, 32 columns of all tokens at a time: xt[chunk][token][32]
  int xt_tokens;            // tokens per chunk of xt
  const float* y;           // tokens x r
  const uint8_t* U;         // r x m, e4m3
  int r;
  float* partial;           // splits x tokens x m
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

// ---- many tokens: bfloat16 matrix cores ----------------------------------------------------------
// O = X~ Dequant^T as a GEMM whose operands are exact in bfloat16: code - zero is an integer of at most
// eight bits, and a float32 x is the sum of its three truncated bfloat16 pieces (8 + 8 + 8 bits), so the
// three products per weight are exact in float32 and only the float32 sums round -- as they do in the
// float32 instruction, which has 1/16 of the rate (three pieces: 1/5.3 of the work).  The group's scale
// is applied to the accumulators where a group ends.
//
// A workgroup takes 32 TT tokens x 128 RT rows of the weight, a wave 32 TT x 32 RT, and walks over chunks of
// 32 columns.  The weight side never touches LDS: lane l of a wave is row l % 32, and half-wave h = l / 32
// takes codes [16 h, 16 h + 16) of the chunk -- the contraction index may be dealt to the lanes in any
// order that both operands share -- so its words come straight from memory and are widened in registers
// (byte conversions, zero subtracted, high halves paired).  X~ lies chunk by chunk, so that the 32 columns of a
// workgroup's tokens are one contiguous piece (row by row, the pieces of all tokens fall on the same few channels of
// the L2); it is read as float32, split while it is staged, and read back as 16-byte fragments; rows of 80 bytes keep those reads free of bank conflicts.
// One barrier per chunk: while chunk c is multiplied, chunk c + 1 is split into the other LDS half and
// chunk c + 2 is on its way from memory.  RT = 2 sets the LDS traffic (six 1 KB reads per twelve MFMAs of a
// wave: half of what the LDS delivers); 64 tokens per workgroup keep 256 registers, two waves per SIMD.
// Bound: the bfloat16 MFMAs (and about nine vector instructions beside each).  The whole call with 16 ranks, against 32-token
// passes on the float32 instruction and an input of two launches: 512 tokens x 4096 x 11008, 3 bits, 1131 -> 167 us;
// 2048 x 11008 x 4096, 4 bits, 4045 -> 540; 4000 x 999 x 1024 2859 -> 65; 32 x 11008 x 4096 82 -> 44; 8 x 4096 x 4096
// 39 -> 20; the distance
// from the float64 product falls from 3.4e-7 to 1.3e-7 of its norm (no sum of code x and zero x of opposite sign).
template <int BITS> struct HalfWords { uint32_t w[BITS == 2 ? 1 : (BITS == 8 ? 4 : 2)]; };

template <int BITS>
__device__ __forceinline__ HalfWords<BITS> load_half_chunk(const uint32_t* __restrict__ base, uint32_t row, int h) {
  const uint32_t off = row + (uint32_t)h * (BITS == 2 || BITS == 3 ? 1u : (BITS == 4 ? 2u : 4u));
  HalfWords<BITS> v;
  if constexpr (BITS == 2) v.w[0] = base[off];
  else if constexpr (BITS == 3) { v.w[0] = base[off]; v.w[1] = base[off + 1]; }   // bits [16 h, 16 h + 48) of these two words
  else if constexpr (BITS == 4) { const uint2 q = *reinterpret_cast<const uint2*>(base + off); v.w[0] = q.x; v.w[1] = q.y; }
  else { const uint4 q = *reinterpret_cast<const uint4*>(base + off); v.w[0] = q.x; v.w[1] = q.y; v.w[2] = q.z; v.w[3] = q.w; }
  return v;
}

// high halves of two floats, the lower one first: two bfloat16 numbers where the low halves are zero
__device__ __forceinline__ uint32_t pair_high(float a, float b) {
  return __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);
}

// codes [8 KS, 8 KS + 8) of a half chunk, minus the group's zero, as bfloat16
template <int BITS, int KS>
__device__ __forceinline__ bf16x8 widen_codes(const HalfWords<BITS>& v, int h, float zero) {
  float f[8];
  if constexpr (BITS == 8) {
#pragma unroll
    for (int j = 0; j < 8; ++j) f[j] = (float)((v.w[2 * KS + (j >> 2)] >> (8 * (j & 3))) & 0xffu);
  } else if constexpr (BITS == 4) {
    const uint32_t even = v.w[KS] & 0x0f0f0f0fu, odd = (v.w[KS] >> 4) & 0x0f0f0f0fu;
#pragma unroll
    for (int j = 0; j < 8; ++j) f[j] = (float)((((j & 1) ? odd : even) >> (8 * (j >> 1))) & 0xffu);
  } else if constexpr (BITS == 2) {
    uint32_t t[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) t[i] = (v.w[0] >> (16 * KS + 2 * i)) & 0x0303u;
#pragma unroll
    for (int j = 0; j < 8; ++j) f[j] = (float)((t[j & 3] >> (8 * (j >> 2))) & 0xffu);
  } else {
    const uint64_t s = (((uint64_t)v.w[1] << 32) | v.w[0]) >> (16 * h);
    const uint32_t b = (uint32_t)(s >> (24 * KS));
#pragma unroll
    for (int j = 0; j < 8; ++j) f[j] = (float)((b >> (3 * j)) & 7u);
  }
  uint4 o;
  o.x = pair_high(f[0] - zero, f[1] - zero);
  o.y = pair_high(f[2] - zero, f[3] - zero);
  o.z = pair_high(f[4] - zero, f[5] - zero);
  o.w = pair_high(f[6] - zero, f[7] - zero);
  return __builtin_bit_cast(bf16x8, o);
}

// The three truncated bfloat16 pieces of two floats, paired.  KEEP_INF: an infinity is its first piece alone, so that its
// products are those of the float32 (otherwise the others are NaN, and so is every sum that it enters).
template <bool KEEP_INF>
__device__ __forceinline__ void split3(float a, float b, uint32_t (&p)[3]) {
  auto rest = [](float v) {
    const float r = v - __uint_as_float(__float_as_uint(v) & 0xffff0000u);
    return KEEP_INF && __builtin_isinf(v) ? 0.f : r;
  };
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    p[i] = pair_high(a, b);
    a = rest(a);
    b = rest(b);
  }
}

// what the scheduler is asked for in a step: after each MFMA one fragment read, as long as there are any, and eight
// vector instructions of the next chunk's preparation
template <int MFMAS, int READS>
__device__ __forceinline__ void tile_sched() {
  if constexpr (MFMAS > 0) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    if constexpr (READS > 0) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);
    tile_sched<MFMAS - 1, (READS > 0 ? READS - 1 : 0)>();
  }
}

constexpr int kTilePitch = 40;   // bfloat16 elements per staged row of 32 columns

struct TilePlan {
  int token_blocks, row_blocks, splits, chunks_per_part;   // splits x KG parts
};

template <int BITS, int TT, int RT, int KG>
__global__ __launch_bounds__(256 * KG, 2) void forward_tile_kernel(ForwardArgs a, int tokens, TilePlan plan) {
  constexpr int kTokens = 32 * TT, kRows = 128 * RT;
  constexpr int E = TT == 1 ? 4 : 8;            // consecutive columns a thread stages: 256 E = 32 kTokens
  __shared__ __attribute__((aligned(16))) uint16_t xs_all[KG][2][3][kTokens][kTilePitch];
  const int part = KG == 1 ? 0 : (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
  const int tid = threadIdx.x & 255, lane = tid & 63, wave = tid >> 6, h = lane >> 5;
  auto& xs = xs_all[part];
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

  const int st_tok = tid / (32 / E), st_col = (tid % (32 / E)) * E;
  const int tok_src = min(tb * kTokens + st_tok, tokens - 1);   // rows past the last token repeat it; not stored
  // per lane: 32-bit offsets that never change; per chunk: one scalar base each
  const uint32_t x_off = (uint32_t)(tok_src - tb * kTokens) * kChunk + (uint32_t)st_col;
  const float* x_base = a.xt + (int64_t)tb * kTokens * kChunk;
  uint32_t row[RT];   // within the workgroup's rows; rows past the last one repeat it, not stored
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
    row[rt] = (uint32_t)min((wave * RT + rt) * 32 + (lane & 31), m - 1 - rb * kRows);
  const uint32_t* packed = a.packed + (int64_t)rb * kRows * BITS;
  const float* scales = a.scales + (int64_t)rb * kRows;
  const uint8_t* zeros = a.zeros + (int64_t)rb * kRows;
  const uint8_t* u_codes = a.U + (int64_t)rb * kRows;

  struct Raw { float x[E]; HalfWords<BITS> w[RT]; float scale[RT]; uint8_t zero[RT]; };
  auto request = [&](Raw& r, int c) {
    c = min(c, c_end - 1);   // issued whatever c: no branch
    const float* xp = x_base + (int64_t)c * a.xt_tokens * kChunk;
#pragma unroll
    for (int i = 0; i < E; i += 4) {
      const float4 v = *reinterpret_cast<const float4*>(xp + x_off + i);
      r.x[i] = v.x; r.x[i + 1] = v.y; r.x[i + 2] = v.z; r.x[i + 3] = v.w;
    }
    const int64_t g = c / gpc;
    const uint32_t* wp = packed + (int64_t)c * m * BITS;
    const float* sp = scales + g * m;
    const uint8_t* zp = zeros + g * m;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      r.w[rt] = load_half_chunk<BITS>(wp, row[rt] * BITS, h);
      r.scale[rt] = sp[row[rt]];
      r.zero[rt] = zp[row[rt]];
    }
  };
  auto stage_x = [&](auto keep_inf, const float (&x)[E], int buf) {
    uint32_t p[E / 2][3];
#pragma unroll
    for (int i = 0; i < E / 2; ++i) split3<decltype(keep_inf)::value>(x[2 * i], x[2 * i + 1], p[i]);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      uint16_t* dst = &xs[buf][k][st_tok][st_col];
      if constexpr (E == 8) *reinterpret_cast<uint4*>(dst) = make_uint4(p[0][k], p[1][k], p[2][k], p[3][k]);
      else *reinterpret_cast<uint2*>(dst) = make_uint2(p[0][k], p[1][k]);
    }
  };

  f32x16 acc[TT][RT], total[TT][RT];
#pragma unroll
  for (int tt = 0; tt < TT; ++tt)
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int r = 0; r < 16; ++r) { acc[tt][rt][r] = 0.f; total[tt][rt][r] = 0.f; }

  auto multiply = [&](const bf16x8 (&b)[2][RT], int buf) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int p = 2; p >= 0; --p)   // the smallest piece first
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
          const bf16x8 av = *reinterpret_cast<const bf16x8*>(&xs[buf][p][tt * 32 + (lane & 31)][16 * h + 8 * ks]);
#pragma unroll
          for (int rt = 0; rt < RT; ++rt)
            acc[tt][rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, b[ks][rt], acc[tt][rt], 0, 0, 0);
        }
  };
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

  Raw raw[2];
  bf16x8 b[2][2][RT];
  float sc[2][RT];
  auto prepare = [&](const Raw& r, int c, int buf, bf16x8 (&bb)[2][RT], float (&s)[RT]) {
    const uint32_t live = c < c_end ? 0xffffffffu : 0u;   // a step past the end multiplies by zero
    float x[E];
#pragma unroll
    for (int i = 0; i < E; ++i) x[i] = __uint_as_float(__float_as_uint(r.x[i]) & live);
    // (an infinite x makes all outputs of its token NaN either way: a row's sum of zero x, were it 0 x, is NaN)
    stage_x(std::false_type{}, x, buf);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const float z = (float)r.zero[rt];
      bb[0][rt] = widen_codes<BITS, 0>(r.w[rt], h, z);
      bb[1][rt] = widen_codes<BITS, 1>(r.w[rt], h, z);
      s[rt] = r.scale[rt];
    }
  };
  request(raw[0], c_begin);
  request(raw[1], c_begin + 1);
  prepare(raw[0], c_begin, 0, b[0], sc[0]);
  int left = gpc - c_begin % gpc;   // chunks until the group ends
  auto step = [&](auto parity, int c) {
    constexpr int P = decltype(parity)::value;
    __syncthreads();
    request(raw[P], c + 2);
    __builtin_amdgcn_sched_barrier(0);
    multiply(b[P], P);
    prepare(raw[P ^ 1], c + 1, P ^ 1, b[P ^ 1], sc[P ^ 1]);
    // the next chunk's conversions go between this chunk's MFMAs, not after them: kept from sinking past the branch
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) asm volatile("" : "+v"(b[P ^ 1][0][rt]), "+v"(b[P ^ 1][1][rt]));
    __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
    tile_sched<6 * TT * RT, 6 * TT - 4>();
    if (--left == 0) { flush(sc[P]); left = gpc; }
  };
  for (int c = c_begin; c < c_begin + plan.chunks_per_part; c += 2) {   // the same count for all waves
    step(std::integral_constant<int, 0>{}, c);
    step(std::integral_constant<int, 1>{}, c + 1);
  }
  flush(sc[1]);   // what is left of the last chunk's group

  // The low-rank part, once: coefficients y (tokens x r) against the e4m3 codes of U, 32 ranks at a time; e4m3
  // is exact in bfloat16, y goes through the same three pieces.
  if (a.r > 0 && split == plan.splits - 1) {
#pragma unroll 1
    for (int k0 = 32 * part; k0 < a.r + 32 * part; k0 += 32 * KG) {   // the same count for all waves
      float yv[E];
#pragma unroll
      for (int i = 0; i < E; ++i) {
        const int k = k0 + st_col + i;
        const float v = a.y[(int64_t)tok_src * a.r + min(k, a.r - 1)];
        yv[i] = k < a.r ? v : 0.f;
      }
      __syncthreads();
      stage_x(std::true_type{}, yv, 0);   // a coefficient past the float32 range makes its products infinite
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          float u[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const int k = k0 + 16 * h + 8 * ks + j;
            const float v = e4m3_to_float(u_codes[(int64_t)min(k, a.r - 1) * m + row[rt]]);
            u[j] = k < a.r ? v : 0.f;
          }
          const uint4 o = make_uint4(pair_high(u[0], u[1]), pair_high(u[2], u[3]), pair_high(u[4], u[5]), pair_high(u[6], u[7]));
          b[0][ks][rt] = __builtin_bit_cast(bf16x8, o);
        }
      __syncthreads();
      multiply(b[0], 0);
    }
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) sc[0][rt] = 1.f;
    flush(sc[0]);
  }

  if constexpr (KG > 1) {   // the second part's sums go to the first through LDS, a tile at a time
    static_assert(KG == 2 && sizeof(xs_all) >= 256 * 16 * sizeof(float), "the exchange reuses the staging area");
    float* ex = reinterpret_cast<float*>(&xs_all[0][0][0][0][0]) + tid;
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

  // accumulator r of a lane is token (r / 4) * 8 + (lane / 32) * 4 + r % 4 of its tile, row lane % 32
  const bool direct = plan.splits == 1;
  float* out = direct ? a.O : a.partial + (int64_t)split * tokens * m;
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

// O[t][row] = sum over the column splits, in order (the last split holds the low-rank part)
__global__ __launch_bounds__(256) void forward_tile_finish_kernel(ForwardArgs a, int tokens, int splits) {
  const int row = blockIdx.x * 256 + threadIdx.x;
  const int t0 = blockIdx.y * 4;
  if (row >= a.m) return;
  float out[4] = {0.f, 0.f, 0.f, 0.f};
  for (int sp0 = 0; sp0 < splits; sp0 += 8) {
    float v[8][4];
#pragma unroll
    for (int k = 0; k < 8; ++k)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int sp = sp0 + k < splits ? sp0 + k : splits - 1;   // issued whatever sp: no branch, no wait
        const int tt = t0 + t < tokens ? t0 + t : tokens - 1;
        v[k][t] = a.partial[((int64_t)sp * tokens + tt) * a.m + row];
      }
#pragma unroll
    for (int k = 0; k < 8; ++k)
#pragma unroll
      for (int t = 0; t < 4; ++t) out[t] += sp0 + k < splits ? v[k][t] : 0.f;
  }
#pragma unroll
  for (int t = 0; t < 4; ++t)
    if (t0 + t < tokens) a.O[(int64_t)(t0 + t) * a.ldo + row] = out[t];
}

constexpr int kFwdRun = 8;            // chunks: the least a column split keeps
constexpr int kPartialTokens = 32;   // the workspace holds partial sums of 32 tokens for every run of 256 columns

template <int BITS, int TT, int KG>
void launch_forward_tile_as(const ForwardArgs& a, int tokens, TilePlan p, hipStream_t st) {
  const int chunks = a.n / kChunk;
  p.chunks_per_part = (int)ceil_div(chunks, p.splits * KG);
  p.splits = (int)ceil_div(chunks, (int64_t)p.chunks_per_part * KG);
  const unsigned grid = 8u * (unsigned)ceil_div((int64_t)p.token_blocks * p.row_blocks * p.splits, 8);
  forward_tile_kernel<BITS, TT, 2, KG><<<grid, 256 * KG, 0, st>>>(a, tokens, p);
  if (p.splits > 1) {
    dim3 gf((unsigned)ceil_div(a.m, 256), (unsigned)ceil_div(tokens, 4));
    forward_tile_finish_kernel<<<gf, 256, 0, st>>>(a, tokens, p.splits);
  }
}

template <int BITS>
void launch_forward_tile(const ForwardArgs& a, int tokens, hipStream_t st) {
  const int chunks = a.n / kChunk;
  const int TT = tokens <= 32 ? 1 : 2;
  TilePlan p{};
  p.token_blocks = (int)ceil_div(tokens, 32 * TT);
  p.row_blocks = (int)ceil_div(a.m, 256);
  const int64_t tiles = (int64_t)p.token_blocks * p.row_blocks;
  // Two waves per SIMD hide each other's loads (one alone waits out about a microsecond per chunk): where the tiles
  // alone give every compute unit two workgroups the columns stay whole; otherwise a workgroup's two halves take half of
  // its columns each (whole call, 16 ranks, 4 bits: 512 tokens x 4096 x 11008 162 us, 177 without; 4000 x 999 x 1024 65 and
  // 68; not at 32 tokens or fewer: 32 x 11008 x 4096 44 and 37, 24 x 11008 x 11008 66 and 54, 8 x 4096 x 4096 19.8 and 19.4),
  // and the columns are split over workgroups until every compute unit has one, as far as the partial sums fit the
  // workspace and a part keeps eight chunks.  Up to 32 tokens the codes' stream is the bound and twice as many
  // workgroups keep more of it in flight (24 x 11008 x 11008 78 -> 66 us, 32 x 11008 x 4096 47 -> 44; 4 x 4096 x 8192
  // loses, 25 -> 29).
  const bool many = tiles >= 512;
  int64_t s = many ? 1 : ceil_div(TT == 1 ? 512 : 256, tiles);
  s = std::min<int64_t>(s, ceil_div(chunks, kFwdRun) * kPartialTokens / tokens);
  s = std::max<int64_t>(1, std::min<int64_t>(s, chunks / kFwdRun));
  p.splits = (int)s;
  const bool halves = !many && chunks / s >= 2;
  if (TT == 1) halves ? launch_forward_tile_as<BITS, 1, 2>(a, tokens, p, st) : launch_forward_tile_as<BITS, 1, 1>(a, tokens, p, st);
  else halves ? launch_forward_tile_as<BITS, 2, 2>(a, tokens, p, st) : launch_forward_tile_as<BITS, 2, 1>(a, tokens, p, st);
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

// One or two tokens always, three or four while their X~ lets two workgroups share a compute unit, go row by row
// (whole call, 4 bits, 16 ranks: 2 x 11008 x 8192 39 us, 54 as tiles; 3 x 11008 x 4096 20.0 and 33.3; 4 x 4096 x 4096
// 18.9 and 19.8; beyond that line 4 x 11008 x 5632 56.3 and 40.5, 4 x 4096 x 8192 32.7 and 29.3, and, three tokens just past
// it, 3 x 11008 x 5632 35.3 and 39.2, 3 x 4096 x 8192 26.5 and 29.3); all others take the tiles.
template <int BITS>
ptq_status launch_forward(const ForwardArgs& a, int tokens, hipStream_t st) {
  if (tokens > 2 && (tokens > 4 || (int64_t)tokens * a.n > 16384)) {
    launch_forward_tile<BITS>(a, tokens, st);
    return PTQ_OK;
  }
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
         align_up((size_t)ceil_div(m, 256) * sizeof(unsigned), 256);   // no kernel uses these: which sizes fit the static array is part of the contract
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
  const PrepArgs prep{X, ldx, (int)tokens, (int)n, perm, b_I, b_H, V, sigma, s, r, xt, y, 0, 0, 0};
  ptq_status rc;
  switch (xdt) {
    case PTQ_F32: rc = launch_forward_prep<PTQ_F32>(prep, st); break;
    case PTQ_BF16: rc = launch_forward_prep<PTQ_BF16>(prep, st); break;
    case PTQ_F64: rc = launch_forward_prep<PTQ_F64>(prep, st); break;
    default: return PTQ_ERR_DTYPE;
  }
  if (rc != PTQ_OK) return rc;
  ForwardArgs a{packed, scales, zeros, (int)m, (int)n, group, xt, (int)tokens, y, U, r, partial, O, ldo};
  switch (bits) {
    case 2: rc = launch_forward<2>(a, (int)tokens, st); break;
    case 3: rc = launch_forward<3>(a, (int)tokens, st); break;
    case 4: rc = launch_forward<4>(a, (int)tokens, st); break;
    case 8: rc = launch_forward<8>(a, (int)tokens, st); break;
    default: return PTQ_ERR_ARG;
  }
  if (rc != PTQ_OK) return rc;
  PTQ_HIP_CHECK_LAUNCH();
  return PTQ_OK;
}

}  // namespace ptq
