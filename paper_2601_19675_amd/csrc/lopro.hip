// LoPRo's pre-conditioning of the layer solve (paper Sec. 3.2): column order (Eq. 5), the
// partial block Walsh-Hadamard rotation of a weight-shaped matrix, R' = R P Q (Eq. 6), its
// way back, Rq Q^T P^T (Eq. 7), and the rotated Hessian H' = Q^T P^T H P Q (Eq. 8).
//
// All of it is memory-bound: every element is read and written once or twice and takes
// log2(b_H) additions on the way.  A row transform stages the row in LDS (so that the
// column gather / scatter never touches HBM at element granularity), and a wave transforms
// 256 consecutive columns at a time, four per lane: two butterfly stages in registers, up to
// six across lanes.  The column direction of H' works on tiles of b_H rows x 32 columns in
// LDS with two register passes of at most sixteen points each.
#include <algorithm>

#include "rotation.h"

namespace ptq {
namespace {

// ---- column order ------------------------------------------------------------------------
constexpr int kOrderSplits = 64;   // row slices whose partial sums are added in a fixed order

// Four columns per thread, eight rows on their way at a time (one column and one row at a time: 35 us for 4096 x 4096
// float32, now 19); ALIGNED: rows on 4-element boundaries, one load per row.
template <int DT, bool ALIGNED>
__global__ __launch_bounds__(256) void abs_colsum_kernel(const void* __restrict__ R, int64_t ldr, int m,
                                                         int n, double* __restrict__ partial) {
  using ST = typename StoredType<DT>::type;
  struct alignas(ALIGNED ? (sizeof(ST) * 4 > 16 ? 16 : sizeof(ST) * 4) : sizeof(ST)) Quad { ST e[4]; };
  const int c = (blockIdx.x * 256 + threadIdx.x) * 4;
  if (c >= n) return;   // n is a multiple of 4 here; otherwise the last thread stops short below
  const ST* col = static_cast<const ST*>(R) + c;
  const int cols = min(4, n - c);
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  constexpr int kRowsAhead = 8;
  for (int r0 = blockIdx.y; r0 < m; r0 += kOrderSplits * kRowsAhead) {
    Quad q[kRowsAhead];
#pragma unroll
    for (int i = 0; i < kRowsAhead; ++i) {
      const int64_t r = min(r0 + i * kOrderSplits, m - 1);   // issued whatever the row: no branch, no wait
      if constexpr (ALIGNED) {
        q[i] = *reinterpret_cast<const Quad*>(col + r * ldr);
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) q[i].e[k] = col[r * ldr + min(k, cols - 1)];
      }
    }
#pragma unroll
    for (int i = 0; i < kRowsAhead; ++i)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const double v = fabs(stored_to_f64<DT>(q[i].e[k]));
        s[k] += r0 + i * kOrderSplits < m ? v : 0.0;
      }
  }
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (k < cols) partial[(int64_t)blockIdx.y * n + c + k] = s[k];
}

__global__ __launch_bounds__(256) void keys_kernel(const double* __restrict__ partial, const double* __restrict__ H,
                                                   int64_t ldh, int m, int n, double* __restrict__ keys) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= n) return;
  double s = 0.0;
  for (int k = 0; k < kOrderSplits; ++k) s += partial[(int64_t)k * n + c];
  const double a = s / (double)m, d = H[(int64_t)c * ldh + c];
  keys[c] = (a != 0.0) ? d / a : (d > 0.0 ? __builtin_inf() : 0.0);
}

// perm[rank] = column, rank = number of columns that come before it (ties: lower index first): of the keys at lower
// indices those that are not behind, of the keys at higher indices those that are ahead.  A lane is a column, a
// workgroup has 64 of them, and each of its sixteen waves compares them with its share of all keys -- read by
// scalar loads, so a comparison and an addition per key are all that a wave issues; the sixteen counts meet in LDS.
// (A sixteenth of the keys per lane out of LDS: 30 us for 4096 columns, now 15.)
constexpr int kRankWaves = 16;
template <bool DESCENDING>
__global__ __launch_bounds__(64 * kRankWaves) void rank_kernel(const double* __restrict__ keys, int n,
                                                               int32_t* __restrict__ perm) {
  __shared__ int counts[kRankWaves][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i0 = blockIdx.x * 64, i = i0 + lane;
  const double ki = keys[min(i, n - 1)];
  auto ahead = [&](double kj) { return DESCENDING ? kj > ki : kj < ki; };
  auto not_behind = [&](double kj) { return DESCENDING ? kj >= ki : kj <= ki; };
  const int share = (n + kRankWaves - 1) / kRankWaves;
  const int j_begin = min(n, wave * share), j_end = min(n, j_begin + share);
  int rank = 0, j = j_begin;
#pragma unroll 8
  for (; j < min(j_end, i0); ++j) rank += not_behind(keys[j]) ? 1 : 0;   // below all of the workgroup's columns
  for (; j < min(j_end, i0 + 64); ++j) {
    const double kj = keys[j];
    rank += (j < i ? not_behind(kj) : ahead(kj)) ? 1 : 0;
  }
#pragma unroll 8
  for (; j < j_end; ++j) rank += ahead(keys[j]) ? 1 : 0;
  counts[wave][lane] = rank;
  __syncthreads();
  if (wave == 0) {
    int total = 0;
#pragma unroll
    for (int w = 0; w < kRankWaves; ++w) total += counts[w][lane];
    if (i < n) perm[total] = i;
  }
}

// ---- row transforms ----------------------------------------------------------------------
// MODE 0:  out[row, c] = sum_c' in[src_row, perm[c']] Q[c', c]     (gather, then rotate)
// MODE 1:  out[row, perm[c]] = sum_c' in[row, c'] Q[c, c']          (rotate, then scatter)
// MODE 2:  MODE 0 for the rows of a symmetric result: what lies left of a rotated row's own block of b_H is left out
// One workgroup per row; the row is staged in LDS in its storage type (MODE 0, 2) resp. as float64
// (MODE 1).  row_perm (MODE 0 and 2, may be null) picks the source row.
// (256 threads, or 1024 when the staged row is so large that only one workgroup fits a CU.)
template <int DT, int MODE>
__global__ __launch_bounds__(1024) void row_rotate_kernel(const void* __restrict__ in, int64_t ldi, int n,
                                                         const int32_t* __restrict__ perm,
                                                         const int32_t* __restrict__ row_perm, int b_I, int b_H,
                                                         double* __restrict__ out, int64_t ldo) {
  extern __shared__ __attribute__((aligned(16))) char rowbuf[];
  using ST = typename StoredType<DT>::type;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nthr = blockDim.x, nwave = nthr >> 6;
  const int row = blockIdx.x;
  const int lg = ilog2(b_H);
  const double scale = 1.0 / sqrt((double)b_H);
  const int nchunk_id = (b_I + 255) / 256;                 // chunks of the identity part
  const int nchunk = nchunk_id + (n - b_I + 255) / 256;    // ... plus those of the rotated part
  if (MODE != 1) {
    const int64_t src = row_perm ? row_perm[row] : row;
    ST* buf = reinterpret_cast<ST*>(rowbuf);
    {
      // 16 bytes at a time where the row allows it
      constexpr int kPer = 16 / (int)sizeof(ST);
      const ST* from = static_cast<const ST*>(in) + src * ldi;
      int c = 0;
      if (reinterpret_cast<uintptr_t>(from) % 16 == 0) {
        c = n / kPer * kPer;
        for (int q = tid * kPer; q < c; q += nthr * kPer) *reinterpret_cast<uint4*>(buf + q) = *reinterpret_cast<const uint4*>(from + q);
      }
      for (c += tid; c < n; c += nthr) buf[c] = from[c];
    }
    __syncthreads();
    // columns below this are another row's mirror image
    const int first = MODE == 2 && row >= b_I ? b_I + (row - b_I) / b_H * b_H : 0;
    for (int k = wave; k < nchunk; k += nwave) {
      const bool ident = k < nchunk_id;
      const int cs = ident ? 256 * k : b_I + 256 * (k - nchunk_id);
      const int ce = ident ? b_I : n;
      if (MODE == 2 && min(cs + 256, ce) <= first) continue;
      const int c = cs + 4 * lane;
      double v[4] = {0.0, 0.0, 0.0, 0.0};
      if (c < ce) {
        const int4 p = *reinterpret_cast<const int4*>(perm + c);
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
      if (c < ce) {
        double* o = out + (int64_t)row * ldo + c;
        *reinterpret_cast<double2*>(o) = double2{v[0], v[1]};
        *reinterpret_cast<double2*>(o + 2) = double2{v[2], v[3]};
      }
    }
  } else {
    double* buf = reinterpret_cast<double*>(rowbuf);
    const double* irow = static_cast<const double*>(in) + (int64_t)row * ldi;
    for (int k = wave; k < nchunk; k += nwave) {
      const bool ident = k < nchunk_id;
      const int cs = ident ? 256 * k : b_I + 256 * (k - nchunk_id);
      const int ce = ident ? b_I : n;
      const int c = cs + 4 * lane;
      double v[4] = {0.0, 0.0, 0.0, 0.0};
      if (c < ce) {
        const double2 a = *reinterpret_cast<const double2*>(irow + c);
        const double2 b = *reinterpret_cast<const double2*>(irow + c + 2);
        v[0] = a.x;
        v[1] = a.y;
        v[2] = b.x;
        v[3] = b.y;
      }
      if (!ident) {
        fwht_chunk(v, lg, lane);
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] *= scale;
      }
      if (c < ce) {
        const int4 p = *reinterpret_cast<const int4*>(perm + c);
        buf[p.x] = v[0];
        buf[p.y] = v[1];
        buf[p.z] = v[2];
        buf[p.w] = v[3];
      }
    }
    __syncthreads();
    for (int c = tid; c < n; c += nthr) out[(int64_t)row * ldo + c] = buf[c];
  }
}

// ---- Hessian -----------------------------------------------------------------------------
// Full symmetric copy of a matrix given by its upper triangle, 32 x 32 tiles through LDS.
__global__ __launch_bounds__(256) void symmetrize_kernel(const double* __restrict__ H, int64_t ldh, int n,
                                                         double* __restrict__ Hs) {
  __shared__ double t[32][33];
  const int I = blockIdx.y, J = blockIdx.x;
  if (I > J) return;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int r = ty; r < 32; r += 8) {
    const int i = I * 32 + r, j = J * 32 + tx;
    double v = 0.0;
    if (i < n && j < n) v = (i <= j) ? H[(int64_t)i * ldh + j] : H[(int64_t)j * ldh + i];
    t[r][tx] = v;
    if (i < n && j < n) Hs[(int64_t)i * n + j] = v;
  }
  __syncthreads();
  if (I == J) return;
  for (int r = ty; r < 32; r += 8) {
    const int i = J * 32 + r, j = I * 32 + tx;
    if (i < n && j < n) Hs[(int64_t)i * n + j] = t[tx][r];
  }
}

// In-place Walsh-Hadamard transform (scaled) down the columns, in blocks of b_H rows starting at
// row b_I: a workgroup takes b_H rows x 32 columns.  With r = 16 a + b inside a block, the first
// pass transforms over b (16 consecutive rows), the second over a (rows 16 apart).
__device__ __forceinline__ void fwht16(double (&x)[16], int lg) {
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    if (s < lg) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        if (!(i & (1 << s))) {
          const double a = x[i], b = x[i | (1 << s)];
          x[i] = a + b;
          x[i | (1 << s)] = a - b;
        }
      }
    }
  }
}

// The result is symmetric: only tiles from a block's own columns on are transformed, and what they hold right of the
// block is also written as the mirror image.  blockIdx.y: the blocks of b_H rows, then the identity rows in pieces of
// at most 256, which are only mirrored.  (All tiles transformed, row pass over all columns: 181 us for the three passes
// at n = 4096, now 145; bound: their bytes.)
__global__ __launch_bounds__(512) void col_rotate_kernel(double* __restrict__ A, int64_t lda, int n, int b_I,
                                                         int b_H) {
  extern __shared__ double tile[];   // [rows][33]
  const int tid = threadIdx.x;
  const int blocks = (n - b_I) / b_H;
  const bool rotated = (int)blockIdx.y < blocks;
  const int r0 = rotated ? b_I + blockIdx.y * b_H : 256 * (blockIdx.y - blocks);
  const int rows = rotated ? b_H : min(256, b_I - r0);
  const int c0 = (rotated ? r0 : b_I) + blockIdx.x * 32;
  if (c0 >= n) return;
  const int lg = ilog2(b_H);
  const double scale = 1.0 / sqrt((double)b_H);
  const int cx = tid & 31;
  for (int r = tid >> 5; r < rows; r += 16)
    tile[r * 33 + cx] = (c0 + cx < n) ? A[(int64_t)(r0 + r) * lda + c0 + cx] : 0.0;
  __syncthreads();
  if (rotated) {
    const int groups = b_H / 16;   // 1 .. 16
    // pass 1: over b (bits 0..3 of the row index), groups x 32 column vectors
    for (int g = tid >> 5; g < groups; g += 16) {
      double x[16];
#pragma unroll
      for (int b = 0; b < 16; ++b) x[b] = tile[(16 * g + b) * 33 + cx];
      fwht16(x, 4);
#pragma unroll
      for (int b = 0; b < 16; ++b) tile[(16 * g + b) * 33 + cx] = x[b];
    }
    __syncthreads();
    // pass 2: over a (bits 4.. of the row index), 16 x 32 column vectors of `groups` points
    for (int b = tid >> 5; b < 16; b += 16) {
      double x[16];
#pragma unroll
      for (int a = 0; a < 16; ++a) x[a] = a < groups ? tile[(16 * a + b) * 33 + cx] : 0.0;
      fwht16(x, lg - 4);
#pragma unroll
      for (int a = 0; a < 16; ++a)
        if (a < groups) tile[(16 * a + b) * 33 + cx] = x[a] * scale;
    }
    __syncthreads();
    for (int r = tid >> 5; r < rows; r += 16)
      if (c0 + cx < n) A[(int64_t)(r0 + r) * lda + c0 + cx] = tile[r * 33 + cx];
  }
  const int mirrored = rotated ? r0 + b_H : b_I;   // columns from here on have their image in other rows
  for (int e = tid; e < 32 * rows; e += 512) {
    const int c = e / rows, r = e - c * rows;
    if (c0 + c >= mirrored && c0 + c < n) A[(int64_t)(c0 + c) * lda + r0 + r] = tile[r * 33 + c];
  }
}

size_t stored_size(ptq_dtype dt) { return dt == PTQ_BF16 ? 2 : (dt == PTQ_F32 ? 4 : 8); }

template <int MODE>
ptq_status launch_row_rotate(const void* in, ptq_dtype dt, int64_t ldi, int64_t rows, int64_t n,
                             const int32_t* perm, const int32_t* row_perm, int b_I, int b_H, double* out,
                             int64_t ldo, hipStream_t st) {
  const size_t lds = (size_t)n * (MODE != 1 ? stored_size(dt) : sizeof(double));
  if (lds > 160 * 1024) return PTQ_ERR_SHAPE;
#define PTQ_ROW_CASE(DT)                                                                                   \
  {                                                                                                        \
    if (!lds_opt_in<row_rotate_kernel<DT, MODE>>(160 * 1024)) return PTQ_ERR_HIP;                          \
    row_rotate_kernel<DT, MODE><<<(unsigned)rows, lds > 40 * 1024 ? 1024 : 256, lds, st>>>(                \
        in, ldi, (int)n, perm, row_perm, b_I, b_H, out, ldo);                                              \
  }
  switch (dt) {
    case PTQ_F32: PTQ_ROW_CASE(PTQ_F32) break;
    case PTQ_BF16: PTQ_ROW_CASE(PTQ_BF16) break;
    case PTQ_F64: PTQ_ROW_CASE(PTQ_F64) break;
    default: return PTQ_ERR_DTYPE;
  }
#undef PTQ_ROW_CASE
  PTQ_HIP_CHECK_LAUNCH();
  return PTQ_OK;
}

}  // namespace

size_t lopro_order_workspace_bytes(int64_t n) {
  return align_up((size_t)(kOrderSplits + 1) * (size_t)n * sizeof(double), 256);
}

size_t lopro_hessian_workspace_bytes(int64_t n) {
  return align_up((size_t)n * (size_t)n * sizeof(double), 256);
}

ptq_status lopro_order_launch(const void* R, ptq_dtype rdt, int64_t ldr, int64_t m, int64_t n, const double* H,
                              int64_t ldh, int descending, int32_t* perm, double* keys, void* ws,
                              hipStream_t st) {
  double* partial = static_cast<double*>(ws);
  double* k = keys ? keys : partial + (size_t)kOrderSplits * n;
  dim3 g((unsigned)ceil_div(n, 1024), kOrderSplits);
  const size_t step = rdt == PTQ_BF16 ? 8 : 16;   // bytes of four elements, at most 16
  const bool aligned = n % 4 == 0 && reinterpret_cast<uintptr_t>(R) % step == 0 && (ldr * (int64_t)stored_size(rdt)) % (int64_t)step == 0;
#define PTQ_COLSUM_CASE(DT)                                                                       \
  if (aligned) abs_colsum_kernel<DT, true><<<g, 256, 0, st>>>(R, ldr, (int)m, (int)n, partial);   \
  else abs_colsum_kernel<DT, false><<<g, 256, 0, st>>>(R, ldr, (int)m, (int)n, partial);
  switch (rdt) {
    case PTQ_F32: PTQ_COLSUM_CASE(PTQ_F32) break;
    case PTQ_BF16: PTQ_COLSUM_CASE(PTQ_BF16) break;
    case PTQ_F64: PTQ_COLSUM_CASE(PTQ_F64) break;
    default: return PTQ_ERR_DTYPE;
  }
#undef PTQ_COLSUM_CASE
  keys_kernel<<<(unsigned)ceil_div(n, 256), 256, 0, st>>>(partial, H, ldh, (int)m, (int)n, k);
  const unsigned gr = (unsigned)ceil_div(n, 64);
  if (descending) rank_kernel<true><<<gr, 64 * kRankWaves, 0, st>>>(k, (int)n, perm);
  else rank_kernel<false><<<gr, 64 * kRankWaves, 0, st>>>(k, (int)n, perm);
  PTQ_HIP_CHECK_LAUNCH();
  return PTQ_OK;
}

ptq_status lopro_rotate_weight_launch(const void* R, ptq_dtype rdt, int64_t ldr, int64_t m, int64_t n,
                                      const int32_t* perm, int b_I, int b_H, double* Rout, int64_t ldo,
                                      hipStream_t st) {
  return launch_row_rotate<0>(R, rdt, ldr, m, n, perm, nullptr, b_I, b_H, Rout, ldo, st);
}

ptq_status lopro_unrotate_weight_launch(const double* Rq, int64_t ldq, int64_t m, int64_t n,
                                        const int32_t* perm, int b_I, int b_H, double* Wout, int64_t ldo,
                                        hipStream_t st) {
  return launch_row_rotate<1>(Rq, PTQ_F64, ldq, m, n, perm, nullptr, b_I, b_H, Wout, ldo, st);
}

ptq_status lopro_rotate_hessian_launch(const double* H, int64_t ldh, int64_t n, const int32_t* perm, int b_I,
                                       int b_H, double* Hout, int64_t ldo, void* ws, hipStream_t st) {
  double* Hs = static_cast<double*>(ws);
  dim3 gs((unsigned)ceil_div(n, 32), (unsigned)ceil_div(n, 32));
  symmetrize_kernel<<<gs, 256, 0, st>>>(H, ldh, (int)n, Hs);
  // rows: Hout[r, :] = (row perm[r] of H, columns gathered by perm) rotated
  ptq_status rc = launch_row_rotate<2>(Hs, PTQ_F64, n, n, n, perm, perm, b_I, b_H, Hout, ldo, st);
  if (rc != PTQ_OK) return rc;
  // columns: H' = Q^T (that)
  if (n > b_I) {
    if (!lds_opt_in<col_rotate_kernel>(256 * 33 * 8)) return PTQ_ERR_HIP;
    dim3 gc((unsigned)ceil_div(n - b_I, 32), (unsigned)((n - b_I) / b_H + ceil_div(b_I, 256)));
    const int rows = std::max(b_H, std::min(b_I, 256));
    col_rotate_kernel<<<gc, 512, (size_t)rows * 33 * sizeof(double), st>>>(Hout, ldo, (int)n, b_I, b_H);
  }
  PTQ_HIP_CHECK_LAUNCH();
  return PTQ_OK;
}

}  // namespace ptq
