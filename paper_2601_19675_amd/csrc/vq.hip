// Vector-quantized form of the column solve: d consecutive columns of a row are assigned one of K
// codebook entries, and the error of the assignment is compensated in the later columns.
//
// Same frame as the scalar solve (quantize.hip): a workgroup owns 16 rows, the lazy update of a block
// of columns is applied left-looking in one float64 MFMA pass over the errors of all earlier columns,
// and inside the block the work goes by 16-column mini-blocks whose errors are pushed onto the later
// tiles with four MFMAs each.  What differs is the walk over a mini-block.  For a group of d columns
// starting at j, with T = U[j:j+d, j:j+d], the loss of entry c for the row's current values w is
// sum_i e_i^2 with e = (w - c) T^-1 taken by forward substitution (the errors the scalar walk would
// make column by column); the entry with the smallest loss is assigned, the lowest index among exactly
// equal ones.  Half a wave works for one row: a lane keeps K / 32 entries in registers for the whole
// walk, evaluates their losses, and the 32 lanes agree on the minimum by data-parallel exchanges (the
// smallest loss first, then the lowest index that has it); the assigned entry comes from a copy of the
// codebook in LDS.  Every lane then knows the group's errors and applies them to the later columns of the
// mini-block itself, so the eight waves walk their two rows each without a barrier between groups.
// Bound: float64 vector instructions of the losses (18 and a selection per entry of 4 weights) and the
// chain from a group's losses to the next group's values.  4096 x 4096, both sides in one run: 256 x 4 3303 -> 2883 us, 64 x 2
// 2441 -> 2276 (before: U and addresses spilled over the walk, an address for every pair read of U, entries tested
// against K one by one; 4.1 ms both with lane permutes through the LDS crossbar, the entry taken out of registers,
// conditional loads, and room for 256 entries in every lane whatever K).  A group of the former takes 1800 cycles.
#include "lazy_update.h"
#include "rotation.h"

namespace ptq {
namespace {

typedef double f64x2 __attribute__((vector_size(16)));

constexpr int kRows = 16;       // rows per workgroup
constexpr int kThreads = 512;
constexpr int kWaves = kThreads / 64;
constexpr int kRowAlign = 96;   // row padding of the error matrix (the scalar solve's workspace layout)
constexpr int kMaxEntries = 256;  // a lane holds SLOTS of them: K <= 32 * SLOTS

struct VqArgs {
  const void* W;
  int64_t ldw;
  int m, n, mpad;
  const double* U;
  int64_t ldu;
  const uint8_t* dead;
  const double* invd;
  double* errT;  // [n][mpad]
  const float* codebook;  // [K][d]
  int K;
  int i1, bw;
  uint8_t* indices;  // [m][n / d]
  double* Wq;
  double* row_err2;
};

__global__ void vq_inv_diag_kernel(const double* __restrict__ U, int64_t ldu, int n, double* invd) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j < n) invd[j] = 1.0 / U[(int64_t)j * ldu + j];
}

// Smallest value over the 32 lanes of a half-wave, in every one of them.
__device__ __forceinline__ double half_wave_min(double v) {
  v = fmin(v, dpp_move<kDppSwapPairs>(v));
  v = fmin(v, dpp_move<kDppSwapHalfQuads>(v));
  v = fmin(v, dpp_move<kDppHalfMirror>(v));
  v = fmin(v, dpp_move<kDppMirror>(v));
  double even, odd;
  lane_pair<false>(v, v, even, odd);
  return fmin(even, odd);
}
__device__ __forceinline__ int half_wave_min(int v) {
  v = min(v, __builtin_amdgcn_update_dpp(0, v, kDppSwapPairs, 0xf, 0xf, true));
  v = min(v, __builtin_amdgcn_update_dpp(0, v, kDppSwapHalfQuads, 0xf, 0xf, true));
  v = min(v, __builtin_amdgcn_update_dpp(0, v, kDppHalfMirror, 0xf, 0xf, true));
  v = min(v, __builtin_amdgcn_update_dpp(0, v, kDppMirror, 0xf, 0xf, true));
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  const u32x2 p = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
  return min((int)p[0], (int)p[1]);
}

// Blocks of 48 to 128 columns: the block of U itself, upper tiles of 16 x 16, is staged in LDS before the walk.  Fetched
// per mini-block it had to be held in registers that the walk does not have: spilled, every request waited for
// the one before, 5000 cycles before and 2500 after the 7400 of a mini-block's walk at 4096 x 4096, 256 x 4.
// (Where a lane holds fewer entries nothing spills and the staging costs 5 % more than it gives, 64 x 2.
// Nor does it pay for blocks of one or two tiles, which ask for the next mini-block's U once or not at all: in a form of
// their own, 4096 x 1024, 256 x 4, blocks of 16 1067 us, staged 1726, and of 32 765, staged 1005; of 48 staged 833, 881.)
template <int NT, int D, int SLOTS, bool RAGGED>
constexpr bool vq_staged() { return NT == 8 && SLOTS * D >= 32 && !RAGGED; }
// tile (r, c), r <= c, in row order; their number; the r and c of number i
__host__ __device__ constexpr int upper_tile(int nt, int r, int c) { return r * nt - r * (r - 1) / 2 + c - r; }
__host__ __device__ constexpr int upper_tiles(int nt) { return nt * (nt + 1) / 2; }
__device__ constexpr int upper_tile_row(int nt, int i) {
  int r = 0;
  while (i >= nt - r) i -= nt - r++;
  return r;
}
__device__ constexpr int upper_tile_column(int nt, int i) {
  const int r = upper_tile_row(nt, i);
  return i - upper_tile(nt, r, r) + r;
}

// RAGGED: a last block whose width is no multiple of 16 (n need only be one of D).  Its last mini-block is walked as far as the
// groups go; nothing past column n of U, the pivots, W or the outputs is read or written, the tiles in LDS are whole.
template <int DT, int NT, int D, int SLOTS, bool RAGGED>
__global__ __launch_bounds__(kThreads) void vq_block_kernel(VqArgs a) {
  extern __shared__ double lds[];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int row0 = blockIdx.x * kRows;
  const int nt = RAGGED ? (a.bw + 15) >> 4 : a.bw >> 4;
  const int pw = RAGGED ? 16 * nt : a.bw;   // columns of the tiles in LDS
  const int sp = pw + 1;  // pitch of the state tile
  auto in_layer = [&](int col) { return RAGGED ? min(col, a.n - 1) : col; };   // a column or row of U past the last: unused
  const double* __restrict__ U = a.U;
  const double* __restrict__ invd = a.invd;
  constexpr int G = 16 / D;  // groups per mini-block

  double* P = lds;                                  // [4][16][pw] partial sums of the lazy update
  double* S = lds;                                  // [16][pw + 1] state tile (aliases P)
  double* Em = lds + 4 * kRows * pw;                // [16 k][16 rows] errors of the mini-block
  double* Qm = Em + 256;                            // [16 k][17] assigned values of the mini-block
  double* Ud = Qm + 272;                            // [2][16][16] diagonal block of U
  double* Id = Ud + 512;                            // [2][16] reciprocal pivots
  double* Cb = Id + 32;                             // [32 SLOTS][D] the codebook
  constexpr bool kStaged = vq_staged<NT, D, SLOTS, RAGGED>();
  double* Ut = Cb + kMaxEntries * D;                // kStaged: [tiles][16][16] the block's upper tiles of U
  double* Ia = Ut + (kStaged ? 256 * upper_tiles(NT) : 0);                 // kStaged: [16 NT] reciprocal pivots
  uint8_t* It = reinterpret_cast<uint8_t*>(Ia + (kStaged ? 16 * NT : 0));  // [16][bw / D] indices of the block

  // ---- phase 1: acc = E[rows, 0:i1] * U[0:i1, block], k split over the waves
  f64x4 acc[NT];
  const bool paired = !RAGGED && lazy_update_paired(nt, a.n, a.ldu, a.mpad);
  auto column_of = [&](int t, int cl) { return paired ? 32 * (t >> 1) + 2 * cl + (t & 1) : 16 * t + cl; };
  lazy_update<NT, kWaves, RAGGED>(U, a.ldu, a.errT, a.mpad, a.n, a.i1, nt, row0, paired, lane, wave, acc, a.bw);
  if (wave >= 4) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
      if (t < nt) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          P[((wave - 4) * kRows + 4 * r + (lane >> 4)) * pw + column_of(t, lane & 15)] = acc[t][r];
      }
  }
  __syncthreads();
  if (wave < 4) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
      if (t < nt) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          P[(wave * kRows + 4 * r + (lane >> 4)) * pw + column_of(t, lane & 15)] += acc[t][r];
      }
  }
  __syncthreads();

  // ---- state tile S = W - (p0 + p1 + p2 + p3), dead channels read as zero; what comes from memory is requested all at
  //      once and whatever the row (loads under a condition wait for each other)
  {
    constexpr int NP = (kRows * 16 * NT + kThreads - 1) / kThreads;
    typename StoredType<DT>::type wraw[NP];
    uint8_t draw[NP];
    int at[NP];   // row * 256 + column of the block
    // (256 threads to a tile of U, two tiles at a time)
    constexpr int NU = kStaged ? (upper_tiles(NT) + 1) / 2 : 1;
    double uraw[NU];
    const int half = __builtin_amdgcn_readfirstlane(tid >> 8);
    auto tile_of = [&](int p, int& tr, int& tc) {
      const int last = upper_tiles(NT) - 1, i1 = 2 * p + 1 < last ? 2 * p + 1 : last;
      tr = half ? upper_tile_row(NT, i1) : upper_tile_row(NT, 2 * p);
      tc = half ? upper_tile_column(NT, i1) : upper_tile_column(NT, 2 * p);
    };
    if constexpr (kStaged) {
#pragma unroll
      for (int p = 0; p < NU; ++p) {
        int tr, tc;
        tile_of(p, tr, tc);
        tr = min(tr, nt - 1);   // (a narrower block: a tile that it has, not stored)
        tc = min(tc, nt - 1);
        uraw[p] = U[(int64_t)(a.i1 + 16 * tr + ((tid >> 4) & 15)) * a.ldu + a.i1 + 16 * tc + (tid & 15)];
      }
    }
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const int e = min(tid + kThreads * p, kRows * a.bw - 1);
      const int r = e / a.bw, c = e - r * a.bw;
      at[p] = r << 8 | c;
      wraw[p] = load_stored<DT>(a.W, (int64_t)min(row0 + r, a.m - 1) * a.ldw + a.i1 + c);
      draw[p] = a.dead ? a.dead[a.i1 + c] : (uint8_t)0;
    }
    double sv[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const int r = at[p] >> 8, c = at[p] & 255;
      const double w = (row0 + r < a.m && draw[p] == 0) ? stored_to_f64<DT>(wraw[p]) : 0.0;
      const double s01 = P[(0 * kRows + r) * pw + c] + P[(1 * kRows + r) * pw + c];
      const double s23 = P[(2 * kRows + r) * pw + c] + P[(3 * kRows + r) * pw + c];
      sv[p] = w - (s01 + s23);
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < NP; ++p)
      if (tid + kThreads * p < kRows * a.bw) S[(at[p] >> 8) * sp + (at[p] & 255)] = sv[p];
    if constexpr (kStaged) {
#pragma unroll
      for (int p = 0; p < NU; ++p) {
        int tr, tc;
        tile_of(p, tr, tc);
        if (tc < nt) Ut[256 * upper_tile(NT, tr, tc) + (tid & 255)] = uraw[p];
      }
      if (tid < a.bw) Ia[tid] = invd[a.i1 + tid];
    } else {
      if (tid < 256) Ud[tid] = U[(int64_t)in_layer(a.i1 + (tid >> 4)) * a.ldu + in_layer(a.i1 + (tid & 15))];
      if (tid < 16) Id[tid] = invd[in_layer(a.i1 + tid)];
    }
    for (int e = tid; e < 32 * SLOTS * D; e += kThreads) Cb[e] = e < a.K * D ? (double)a.codebook[e] : 0.0;
  }
  __syncthreads();

  // ---- phase 2: 16-column mini-blocks; half a wave walks one row
  // this lane's codebook entries, k = l32 + 32 s, in registers from here on (after the lazy update, whose
  // accumulators need the room)
  const int l32 = lane & 31;
  // (one that does not exist is infinitely far away: its loss is no smaller than any)
  double cb[SLOTS][D];
#pragma unroll
  for (int s = 0; s < SLOTS; ++s)
#pragma unroll
    for (int i = 0; i < D; ++i) cb[s][i] = l32 + 32 * s < a.K ? Cb[(l32 + 32 * s) * D + i] : __builtin_inf();
  const int r = 2 * wave + (lane >> 5);   // the row of this half-wave
  double err2 = 0.0;
  constexpr int kUpd = (NT + kWaves - 1) / kWaves;
  const int gpb = a.bw / D;               // groups per block (pitch of the index tile)
  for (int mb = 0; mb < nt; ++mb) {
    const int c0 = 16 * mb;
    const int gcol = a.i1 + c0;
    const int buf = mb & 1;
    double ud_next = 0.0, id_next = 0.0;
    double ub[kUpd][4];
    if constexpr (!kStaged) {
      if (mb + 1 < nt) {
        if (tid < 256) ud_next = U[(int64_t)in_layer(gcol + 16 + (tid >> 4)) * a.ldu + in_layer(gcol + 16 + (tid & 15))];
        if (tid < 16) id_next = invd[in_layer(gcol + 16 + tid)];
      }
#pragma unroll
      for (int q = 0; q < kUpd; ++q) {
        const int t = mb + 1 + wave + kWaves * q;
        const int tc = t < nt ? t : nt - 1;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
          ub[q][kk] = U[(int64_t)in_layer(gcol + 4 * kk + (lane >> 4)) * a.ldu + in_layer(a.i1 + 16 * tc + (lane & 15))];
      }
    }
    {
      const double* ud = kStaged ? Ut + 256 * upper_tile(NT, mb, mb) : Ud + buf * 256;
      const double* id = kStaged ? Ia + 16 * mb : Id + buf * 16;
      // entries [from, to) right of column c of row `row` of the block into x[from ..], 16 bytes at a time: the offset of an
      // 8-byte pair read ends at 2 KB, and most of the rows would take an address of their own
      auto fetch_row = [&](double* x, int from, int to, int row, int c) {
        if constexpr (D % 2 == 0) {
#pragma unroll
          for (int k = from & ~1; k < to; k += 2) {
            const f64x2 two = *reinterpret_cast<const f64x2*>(ud + row * 16 + c + k);
            if (k >= from) x[k] = two[0];
            x[k + 1] = two[1];
          }
        } else {
#pragma unroll
          for (int k = from; k < to; ++k) x[k] = ud[row * 16 + c + k];
        }
      };
      double w[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) w[j] = S[r * sp + c0 + j];
#pragma unroll
      for (int g = 0; g < G; ++g) {
        if (RAGGED && c0 + g * D >= a.bw) continue;
        __builtin_amdgcn_sched_barrier(0);   // a group's LDS reads stay in it: all groups' together do not fit the registers
        // the group's triangle of U and its reciprocal pivots
        double T[D][D], inv[D];
#pragma unroll
        for (int i = 0; i < D; ++i) {
          inv[i] = id[g * D + i];
          fetch_row(T[i], i + 1, D, g * D + i, g * D);
        }
        // losses of this lane's entries, ascending index: a later entry wins only if strictly smaller
        double best = __builtin_inf();
        int bidx = 0x7fffffff;
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
          const int k = l32 + 32 * s;
          double rem[D], loss = 0.0;
#pragma unroll
          for (int i = 0; i < D; ++i) rem[i] = w[g * D + i] - cb[s][i];
#pragma unroll
          for (int i = 0; i < D; ++i) {
            const double e = rem[i] * inv[i];
#pragma unroll
            for (int kx = i + 1; kx < D; ++kx) rem[kx] = fma(-e, T[i][kx], rem[kx]);
            loss = fma(e, e, loss);
          }
          const bool take = loss < best;
          best = take ? loss : best;
          bidx = take ? k : bidx;
        }
        {
          const double smallest = half_wave_min(best);
          bidx = half_wave_min(best == smallest ? bidx : 0x7fffffff);
        }
        // every lane of the half-wave now holds the assigned index (one past the codebook if no loss was a number)
        double q[D], e[D];
        {
          const int entry = bidx < 32 * SLOTS ? bidx : 31;
#pragma unroll
          for (int i = 0; i < D; ++i) q[i] = Cb[entry * D + i];
        }
        {
          double rem[D];
#pragma unroll
          for (int i = 0; i < D; ++i) rem[i] = w[g * D + i] - q[i];
#pragma unroll
          for (int i = 0; i < D; ++i) {
            e[i] = rem[i] * inv[i];
#pragma unroll
            for (int kx = i + 1; kx < D; ++kx) rem[kx] = fma(-e[i], T[i][kx], rem[kx]);
          }
        }
        // the group's errors onto the later columns of the mini-block
        {
          double u[16];
#pragma unroll
          for (int i = 0; i < D; ++i) {   // (per column the rows in order)
            fetch_row(u, (g + 1) * D, 16, g * D + i, 0);
#pragma unroll
            for (int c = (g + 1) * D; c < 16; ++c) w[c] = fma(-e[i], u[c], w[c]);
          }
        }
        if (l32 == 0) {
#pragma unroll
          for (int i = 0; i < D; ++i) {
            Em[(g * D + i) * kRows + r] = e[i];
            Qm[(g * D + i) * 17 + r] = q[i];
            err2 = fma(e[i], e[i], err2);
          }
          It[r * gpb + mb * G + g] = (uint8_t)bidx;
        }
      }
    }
    // (what follows computes its addresses anew: kept over the walk they are spilled, and a reload waits for the stores
    // of the mini-block before)
    int ln = lane, tl = tid;
    if constexpr (kStaged) asm volatile("" : "+v"(ln), "+v"(tl));
    if constexpr (kStaged) {
#pragma unroll
      for (int q = 0; q < kUpd; ++q) {
        const int t = min(mb + 1 + wave + kWaves * q, nt - 1);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) ub[q][kk] = Ut[256 * upper_tile(NT, mb, t) + (4 * kk + (ln >> 4)) * 16 + (ln & 15)];
      }
    }
    __syncthreads();
    // push the 16 new errors onto the later tiles of the block
#pragma unroll
    for (int q = 0; q < kUpd; ++q) {
      const int t = mb + 1 + wave + kWaves * q;
      if (t < nt) {
        f64x4 d = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          const double av = Em[(4 * kk + (ln >> 4)) * kRows + (ln & 15)];
          d = __builtin_amdgcn_mfma_f64_16x16x4f64(av, ub[q][kk], d, 0, 0, 0);
        }
        double sv[4];
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) sv[rr] = S[(4 * rr + (ln >> 4)) * sp + 16 * t + (ln & 15)];
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) S[(4 * rr + (ln >> 4)) * sp + 16 * t + (ln & 15)] = sv[rr] - d[rr];
      }
    }
    if (tl >= 256) {
      const int e = tl - 256;
      if (!RAGGED || gcol + (e >> 4) < a.n) a.errT[(int64_t)(gcol + (e >> 4)) * a.mpad + row0 + (e & 15)] = Em[e];
      const int rr = e >> 4, j = e & 15;
      if (a.Wq && row0 + rr < a.m && (!RAGGED || gcol + j < a.n)) a.Wq[(int64_t)(row0 + rr) * a.n + gcol + j] = Qm[j * 17 + rr];
    }
    if (!kStaged && mb + 1 < nt) {
      if (tid < 256) Ud[(buf ^ 1) * 256 + tid] = ud_next;
      if (tid < 16) Id[(buf ^ 1) * 16 + tid] = id_next;
    }
    __syncthreads();
  }

  // ---- outputs of the block
  const int ng = a.n / D;
  for (int e = tid; e < kRows * gpb; e += kThreads) {
    const int rr = e / gpb, c = e - rr * gpb;
    if (row0 + rr < a.m) a.indices[(int64_t)(row0 + rr) * ng + a.i1 / D + c] = It[rr * gpb + c];
  }
  if (a.row_err2 && (lane & 31) == 0 && row0 + r < a.m) {
    if (a.i1 == 0)
      a.row_err2[row0 + r] = err2;
    else
      a.row_err2[row0 + r] += err2;
  }
}

// (staged: the block of U, for blocks of nt tiles at most)
size_t vq_lds_bytes(int bw, int d, int staged_nt) {
  const int staged = staged_nt ? 256 * upper_tiles(staged_nt) + 16 * staged_nt : 0;
  return (size_t)(4 * kRows * bw + 256 + 272 + 512 + 32 + kMaxEntries * d + staged) * sizeof(double) + (size_t)kRows * bw;
}

template <int DT, int NT, int D, int SLOTS, bool RAGGED = false>
ptq_status vq_launch_block(const VqArgs& a, hipStream_t st) {
  if (!lds_opt_in<vq_block_kernel<DT, NT, D, SLOTS, RAGGED>>((int)vq_lds_bytes(16 * NT, D, vq_staged<NT, D, SLOTS, RAGGED>() ? NT : 0))) return PTQ_ERR_HIP;
  const size_t lds = vq_lds_bytes((a.bw + 15) / 16 * 16, D, vq_staged<NT, D, SLOTS, RAGGED>() ? NT : 0);
  vq_block_kernel<DT, NT, D, SLOTS, RAGGED><<<(unsigned)ceil_div(a.m, kRows), kThreads, lds, st>>>(a);
  return PTQ_OK;
}

template <int DT, int D, int SLOTS>
ptq_status vq_run_blocks_with(VqArgs a, int block, hipStream_t st) {
  for (int i1 = 0; i1 < a.n; i1 += block) {
    a.i1 = i1;
    a.bw = (a.n - i1 < block) ? a.n - i1 : block;
    // (one form of the ragged kernel, for all widths and codebooks: it takes a layer's last block only)
    if constexpr (vq_staged<8, D, SLOTS, false>()) {
      if (a.bw == 16 || a.bw == 32) {
        const ptq_status rc = vq_launch_block<DT, 2, D, SLOTS>(a, st);
        if (rc != PTQ_OK) return rc;
        continue;
      }
    }
    const ptq_status rc = a.bw % 16 != 0 ? vq_launch_block<DT, 16, D, kMaxEntries / 32, true>(a, st)
                          : a.bw <= 128  ? vq_launch_block<DT, 8, D, SLOTS>(a, st)
                                         : vq_launch_block<DT, 16, D, SLOTS>(a, st);
    if (rc != PTQ_OK) return rc;
  }
  return PTQ_OK;
}

template <int DT, int D>
ptq_status vq_run_blocks(const VqArgs& a, int block, hipStream_t st) {
  return a.K <= 64 ? vq_run_blocks_with<DT, D, 2>(a, block, st) : vq_run_blocks_with<DT, D, 8>(a, block, st);
}

template <int DT>
ptq_status vq_run_dim(const VqArgs& a, int d, int block, hipStream_t st) {
  switch (d) {
    case 1: return vq_run_blocks<DT, 1>(a, block, st);
    case 2: return vq_run_blocks<DT, 2>(a, block, st);
    case 4: return vq_run_blocks<DT, 4>(a, block, st);
    default: return PTQ_ERR_ARG;
  }
}

}  // namespace

ptq_status quantize_vq_launch(const void* W, ptq_dtype wdt, int64_t ldw, int64_t m, int64_t n, const double* U,
                              int64_t ldu, const uint8_t* dead_mask, const float* codebook, int entries, int dim,
                              int block, uint8_t* indices, double* Wq, double* row_err2, void* ws, size_t ws_bytes,
                              hipStream_t st) {
  if (m == 0 || n == 0) return PTQ_OK;
  if (ws_bytes < quantize_workspace_bytes(m, n)) return PTQ_ERR_WORKSPACE;
  VqArgs a;
  a.W = W;
  a.ldw = ldw;
  a.m = (int)m;
  a.n = (int)n;
  a.mpad = (int)(ceil_div(m, kRowAlign) * kRowAlign);
  a.U = U;
  a.ldu = ldu;
  a.dead = dead_mask;
  a.errT = static_cast<double*>(ws);
  a.invd = reinterpret_cast<double*>(static_cast<char*>(ws) + align_up((size_t)n * (size_t)a.mpad * sizeof(double), 256));
  a.codebook = codebook;
  a.K = entries;
  a.i1 = 0;
  a.bw = 0;
  a.indices = indices;
  a.Wq = Wq;
  a.row_err2 = row_err2;
  vq_inv_diag_kernel<<<(unsigned)ceil_div(n, 256), 256, 0, st>>>(U, ldu, (int)n, const_cast<double*>(a.invd));
  PTQ_HIP_CHECK_LAUNCH();
  ptq_status rc;
  switch (wdt) {
    case PTQ_F32: rc = vq_run_dim<PTQ_F32>(a, dim, block, st); break;
    case PTQ_BF16: rc = vq_run_dim<PTQ_BF16>(a, dim, block, st); break;
    case PTQ_F64: rc = vq_run_dim<PTQ_F64>(a, dim, block, st); break;
    default: return PTQ_ERR_DTYPE;
  }
  if (rc != PTQ_OK) return rc;
  PTQ_HIP_CHECK_LAUNCH();
  return PTQ_OK;
}

}  // namespace ptq
