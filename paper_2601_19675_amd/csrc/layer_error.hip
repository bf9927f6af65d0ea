// Relative layer error  sqrt( tr(D H D^T) / tr(W H W^T) ),  D = W - Wq.
//
// H is symmetric and only its upper triangle is stored, so each quadratic form
// is evaluated as  sum_ij A_ij * (A Hu)_ij  with
//     Hu(k,j) = 2 H(k,j) for k < j,  H(k,k) for k == j,  0 for k > j,
// which reads every stored entry once in its coalesced direction and halves the
// work of the float64 MFMA GEMM (the k range of a column tile stops at its last
// column).  Each workgroup reduces its tile to one number; a final
// single-workgroup kernel adds the tile sums in index order.
//
// Two forms of the same sum.  Weights stored in float64 take the float64 MFMA GEMM.  Weights
// stored in float32 or bfloat16 take the bfloat16-split one: D, W and Hu are rounded to float32
// once (W in bfloat16 is exact) and kept as three bfloat16 pieces each, two in large layers (kTwoPiecesFrom);
// the piece products and the running sums over k are float32 on the matrix cores, and everything
// from the tile's sum_ij A_ij T_ij on is float64.  The roundings are unbiased and independent, so they
// average out over the m n terms of the trace.  Two pieces go in tiles of 256 x 128 where there are enough of them.
#include "dgemm.h"
#include "lds_dma.h"

namespace ptq {
namespace {

constexpr int TM = 2, TN = 4;  // 64 x 128 tile: two workgroups (8 waves) per CU keep the f64 matrix pipe fuller
using Tile = DgemmTile<TM, TN>;

struct ErrArgs {
  const double* A2;  // [2][m][n]: D = W - Wq, then W, both widened to float64
  int m, n;
  const double* H;
  int64_t ldh;
  double* partial;  // [2][tiles]
};

// D = W - Wq next to W itself, both dense, so that the GEMM streams two plain matrices.
__global__ __launch_bounds__(256) void widen_kernel(const double* __restrict__ W, int64_t ldw,
                                                    const double* __restrict__ Wq, int m, int n,
                                                    double* __restrict__ A2) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= (int64_t)m * n) return;
  const int i = (int)(e / n), k = (int)(e - (int64_t)i * n);
  const double w = W[(int64_t)i * ldw + k];
  A2[e] = w - Wq[e];
  A2[(int64_t)m * n + e] = w;
}

__global__ __launch_bounds__(256, 3) void quad_form_kernel(ErrArgs a) {   // three workgroups per CU fit in LDS
  extern __shared__ double smem[];
  __shared__ double red[256];
  // column tiles have k ranges proportional to their index: the widest are dispatched
  // first (blockIdx.y is the slow grid index), the two quadratic forms share blockIdx.x
  const int nrt = gridDim.x >> 1;
  const int z = blockIdx.x / nrt;
  const int rt = blockIdx.x - z * nrt;
  const int ct = gridDim.y - 1 - blockIdx.y;
  const int i0 = rt * Tile::BM, j0 = ct * Tile::BN;
  const int j1 = min(j0 + Tile::BN, a.n);
  const int i1 = min(i0 + Tile::BM, a.m);
  const double* Az = a.A2 + (int64_t)z * a.m * a.n;
  f64x4 acc[TM][TN];
  dgemm_zero(acc);
  dgemm_mainloop<TM, TN, true, false>(
      acc, DView{Az + (int64_t)i0 * a.n, a.n, 1}, DgemmIdentity{},
      // H below the diagonal is read (it is valid memory) and discarded
      DView{a.H + j0, 1, a.ldh},
      [&](double h, int k, int j) { return k == j0 + j ? h : (k < j0 + j ? 2.0 * h : 0.0); },
      i1 - i0, j1 - j0, 0, j1, smem);
  double s = 0.0;
  dgemm_foreach(acc, [&](int i, int j, double v) {
    const bool ok = (i0 + i < a.m) & (j0 + j < a.n);
    const double d = Az[ok ? (int64_t)(i0 + i) * a.n + j0 + j : 0];
    s = fma(v, ok ? d : 0.0, s);
  });
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0)
    a.partial[((int64_t)z * nrt + rt) * gridDim.y + ct] = red[0];
}

// ---------------------------------------------------------------- bfloat16-split form
constexpr int kT = 128;         // tile edge: four waves, 64 x 64 each (2 x 2 tiles of the 32 x 32 x 16 MFMA)

// A number rounded to P bfloat16 pieces (8 significant bits each, each remainder taken after rounding
// to nearest) keeps 8 P significant bits, and the product of two bfloat16 numbers is exact in
// float32.  So A Hu is the sum of the piece products A_a Hu_b; those with a + b < P carry everything
// down to 2^(-8 P) of a term, the others are below what the pieces resolve.  They run on the bfloat16
// 32 x 32 x 16 MFMA, accumulate in float32, smallest pieces first.  W stored in bfloat16 is one piece.
// Three pieces are float32 arithmetic (six products for tr(D H D^T), three for tr(W H W^T) with W in
// bfloat16; the traces agree with the float64 definition to 1e-8, 3e-7 at worst).  With two pieces
// (three and two products, 0.56 of the matrix-core work) every term is off by up to 2^-16 of itself,
// unbiased and independent from term to term, and a trace adds m n of them: measured against the
// float64 oracle on layers of 1e5 .. 4.5e7 entries the traces differ by 3e-7 .. 1e-6 relative and the
// relative layer error by at most 1e-7, where the required agreement is 1e-4.  That rests on the
// averaging, so layers of fewer than kTwoPiecesFrom entries (where the time does not matter) take three.
constexpr int kMaxPieces = 3;
constexpr int64_t kTwoPiecesFrom = 65536;
constexpr int kSK = 32;        // k-tile of the split form
constexpr int kSP = kSK + 8;   // LDS pitch in elements: 80-byte rows keep the 16-byte fragment reads apart

__device__ __forceinline__ uint16_t bf16_rne(float x) {
  uint32_t u = __float_as_uint(x);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf16_val(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
template <int P>
__device__ __forceinline__ void split(float x, uint16_t (&p)[P]) {
  float r = x;
#pragma unroll
  for (int q = 0; q < P; ++q) {
    p[q] = bf16_rne(r);
    r -= bf16_val(p[q]);
  }
}

struct SplitArgs {
  const uint16_t* D;   // [P][mp][np]: D = W - Wq as bfloat16 pieces; zero outside m x n
  const uint16_t* W;   // [1 or P][mp][np]: W likewise
  const uint16_t* HuT; // [P][np (j)][np (k)]: Hu transposed, as pieces; zero for k > j and outside n x n
  int mp, np;
  double* partial;     // [2][tiles]: the tile sums of tr(D H D^T), then those of tr(W H W^T)
};

constexpr int kWideM = 256;   // rows of a tile of the wide form
constexpr int kSlab = 16;            // rows of tiles that are worked on together; a multiple of 8

// D and W as bfloat16 pieces, four consecutive k per thread
template <int DT, int P>
__global__ __launch_bounds__(256) void split_weights_kernel(const void* __restrict__ W, int64_t ldw,
                                                            const double* __restrict__ Wq, int m, int n, int mp, int np,
                                                            uint16_t* __restrict__ Dp, uint16_t* __restrict__ Wp) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q >= (int64_t)mp * np / 4) return;
  const int i = (int)(q / (np / 4)), k0 = (int)(q - (int64_t)i * (np / 4)) * 4;
  uint16_t d[4][P], w[4][P];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const bool ok = i < m && k0 + c < n;
    const double wv = ok ? load_as_f64<DT>(W, (int64_t)i * ldw + k0 + c) : 0.0;
    const double qv = ok ? Wq[(int64_t)i * n + k0 + c] : 0.0;
    split((float)(wv - qv), d[c]);
    split((float)wv, w[c]);
  }
  const int64_t plane = (int64_t)mp * np, at = (int64_t)i * np + k0;
#pragma unroll
  for (int p = 0; p < P; ++p) {
    *reinterpret_cast<ushort4*>(Dp + p * plane + at) = ushort4{d[0][p], d[1][p], d[2][p], d[3][p]};
    if (DT != PTQ_BF16 || p == 0)
      *reinterpret_cast<ushort4*>(Wp + p * plane + at) = ushort4{w[0][p], w[1][p], w[2][p], w[3][p]};
  }
}

// Hu transposed, as pieces: 32 x 32 tiles through LDS so that both the reads of H and the writes run along rows
template <int P>
__global__ __launch_bounds__(256) void split_hu_kernel(const double* __restrict__ H, int64_t ldh, int n, int np,
                                                       uint16_t* __restrict__ HuT) {
  __shared__ uint16_t t[P][32][33];
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const int j0 = blockIdx.x * 32, k0 = blockIdx.y * 32;
#pragma unroll
  for (int rr = 0; rr < 4; ++rr) {
    const int k = k0 + ty + 8 * rr, j = j0 + tx;
    const bool ok = k < n && j < n && k <= j;
    const double h = ok ? H[(int64_t)k * ldh + j] : 0.0;
    uint16_t p[P];
    split((float)(k == j ? h : 2.0 * h), p);
#pragma unroll
    for (int q = 0; q < P; ++q) t[q][ty + 8 * rr][tx] = p[q];
  }
  __syncthreads();
  const int64_t plane = (int64_t)np * np;
#pragma unroll
  for (int rr = 0; rr < 4; ++rr) {
    const int j = j0 + ty + 8 * rr, k = k0 + tx;
#pragma unroll
    for (int q = 0; q < P; ++q) HuT[q * plane + (int64_t)j * np + k] = t[q][tx][ty + 8 * rr];
  }
}

// ND pieces of D and NW pieces of W against the NH pieces of Hu: both traces in one pass over Hu
// (<P, 1, P>: W stored in bfloat16), or one trace per slice of the grid (<P, 0, P>)
template <int ND, int NW, int NH>
__global__ __launch_bounds__(256) void quad_form_split_kernel(SplitArgs a) {
  extern __shared__ uint16_t sm[];   // [2 stages][ND + NW + NH pieces][128 rows][kSP]
  __shared__ double red[2][4];
  constexpr int NA = ND + NW, NP = NA + NH;
  constexpr int kPiece = kT * kSP, kStage = NP * kPiece;
  // the widest column tiles first (blockIdx.y is the slow grid index)
  const int rt = blockIdx.x, ct = gridDim.y - 1 - blockIdx.y;
  const int i0 = rt * kT, j0 = ct * kT;
  const int kend = j0 + kT;   // beyond it Hu is zero; a multiple of 128
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int64_t planeA = (int64_t)a.mp * a.np, planeB = (int64_t)a.np * a.np;

  // a piece's 128 x 32 tile is 512 chunks of 16 bytes: two per thread.  Two register sets: a tile's
  // loads are issued three k-tiles ahead and have two whole k-tiles of MFMAs to arrive (one k-tile
  // of the bfloat16 MFMA is too short to cover the latency of a load from L2)
  const int lr = tid >> 2, lk = (tid & 3) * 8;
  const int64_t arow = (int64_t)(i0 + lr) * a.np + lk;
  const uint16_t* gb = a.HuT + (int64_t)(j0 + lr) * a.np + lk;
  // with NW = 0 the two traces are two slices of the grid: the same products on the pieces of D and on those of W
  const uint16_t* first = NW == 0 && blockIdx.z ? a.W : a.D;
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));   // a native vector: stays in registers
  u32x4 reg[2][NP][2];
  auto fetch = [&](auto set, int k0) {
    constexpr int S = decltype(set)::value;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const uint16_t* g = p < ND ? first + p * planeA + arow : (p < NA ? a.W + (p - ND) * planeA + arow : gb + (p - NA) * planeB);
      reg[S][p][0] = *reinterpret_cast<const u32x4*>(g + k0);
      reg[S][p][1] = *reinterpret_cast<const u32x4*>(g + (int64_t)64 * a.np + k0);
    }
  };
  auto stash = [&](auto set, int stage) {
    constexpr int S = decltype(set)::value;
    uint16_t* st = sm + stage * kStage;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      *reinterpret_cast<u32x4*>(st + p * kPiece + lr * kSP + lk) = reg[S][p][0];
      *reinterpret_cast<u32x4*>(st + p * kPiece + (lr + 64) * kSP + lk) = reg[S][p][1];
    }
  };

  constexpr int kForms = 1 + (NW > 0);
  f32x16 acc[kForms][2][2];
#pragma unroll
  for (int f = 0; f < kForms; ++f)
#pragma unroll
    for (int tm = 0; tm < 2; ++tm)
#pragma unroll
      for (int tn = 0; tn < 2; ++tn)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[f][tm][tn][r] = 0.f;

  // One k-tile: the products of the tile in LDS stage `stage`, with the next tile's way into the other stage
  // (registers of `set` -> LDS, then the loads of tile knext into the same registers) issued between them.
  // A wave is alone on its SIMD, so nothing hides what it waits for but its own MFMAs: the fragments of the
  // second k-step are read while the first k-step's products run, the LDS stores go out between them too,
  // and the global loads go out between the products of the second k-step.  Only the first k-step's
  // fragment reads, right after the barrier, are exposed.  The order is asked of the scheduler explicitly.
  struct Frags {
    bf16x8 a[NA][2], b[NH][2];
  };
  auto read_frags = [&](const uint16_t* st, int ks, Frags& f) {
    // fragment of a 32-row strip: lane l holds row l % 32, k = 8 (l / 32) .. + 7 of the 16-wide k-step
    const int fo = (lane & 31) * kSP + ks * 16 + (lane >> 5) * 8;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
#pragma unroll
      for (int p = 0; p < NA; ++p)
        f.a[p][t] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(st + p * kPiece + (wm * 64 + t * 32) * kSP + fo));
#pragma unroll
      for (int p = 0; p < NH; ++p)
        f.b[p][t] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(st + (NA + p) * kPiece + (wn * 64 + t * 32) * kSP + fo));
    }
  };
  // piece pa of an operand with piece pb of Hu for pa + pb < NH, the smallest products first
  auto multiply = [&](const Frags& f) {
#pragma unroll
    for (int order = NH - 1; order >= 0; --order)
#pragma unroll
      for (int p = 0; p < NA; ++p) {
        const int fr = p >= ND ? 1 : 0;   // which trace the piece belongs to
        const int pa = p < ND ? p : p - ND;
        const int pb = order - pa;
        if (pb < 0 || pb >= NH) continue;
#pragma unroll
        for (int tm = 0; tm < 2; ++tm)
#pragma unroll
          for (int tn = 0; tn < 2; ++tn)
            acc[fr][tm][tn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[p][tm], f.b[pb][tn], acc[fr][tm][tn], 0, 0, 0);
      }
  };
  constexpr int kFull = NH * (NH + 1) / 2;   // products of an operand that has all its pieces
  constexpr int kMfma = 4 * ((ND ? kFull : 0) + (NW == NH ? kFull : (NW == 1 ? NH : 0)));   // MFMAs of one k-step
  constexpr int kMem = 2 * NP;                         // fragment reads = LDS stores = loads of a k-tile
  constexpr int kPer = kMfma / kMem, kRest = kMfma - kPer * kMem;   // MFMAs between two memory instructions
  static_assert(ND > 0, "D or, in the second slice, W in its place");
  static_assert(kSK == 32 && kPer >= 1, "two k-steps per tile; at least one MFMA between memory instructions");
  auto tile = [&](auto stage_c, auto set, int knext) {
    constexpr int STAGE = decltype(stage_c)::value;
    const uint16_t* st = sm + STAGE * kStage;
    Frags f0, f1;
    __builtin_amdgcn_sched_barrier(0);
    read_frags(st, 0, f0);
    read_frags(st, 1, f1);
    stash(set, STAGE ^ 1);
    multiply(f0);
    fetch(set, knext);
    multiply(f1);
    // the first k-step's fragments; then per kPer MFMAs one fragment read of the second k-step and one LDS
    // store; then per kPer MFMAs one global load
    __builtin_amdgcn_sched_group_barrier(0x100, kMem, 0);
#pragma unroll
    for (int i = 0; i < kMem; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, kPer, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
    }
    if constexpr (kRest > 0) __builtin_amdgcn_sched_group_barrier(0x008, kRest, 0);
#pragma unroll
    for (int i = 0; i < kMem; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, kPer, 0);
      __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
    }
    if constexpr (kRest > 0) __builtin_amdgcn_sched_group_barrier(0x008, kRest, 0);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
  };
  using Set0 = std::integral_constant<int, 0>;
  using Set1 = std::integral_constant<int, 1>;
  using Stage0 = std::integral_constant<int, 0>;
  using Stage1 = std::integral_constant<int, 1>;

  // kend is a multiple of 128: an even number (at least four) of k-tiles.  The loop body has no
  // branch: a fetch beyond the last k-tile reads the last one again and a stash after the last
  // products fills a stage nobody reads.  With conditional fetches the compiler cannot count the
  // outstanding loads across the back edge and waits for all of them before every stash; as it
  // stands it waits for all but the newest set, and a tile's loads have two k-tiles to arrive.
  // (The prologue issues its loads in the loop's order, set 1 before the second set 0, and the
  // scheduling barriers keep it so: the wait counts at the loop head are the worse of the two ways in.)
  const int klast = kend - kSK;
  fetch(Set0{}, 0);
  __builtin_amdgcn_sched_barrier(0);
  fetch(Set1{}, kSK);
  __builtin_amdgcn_sched_barrier(0);
  stash(Set0{}, 0);
  __builtin_amdgcn_sched_barrier(0);
  fetch(Set0{}, 2 * kSK);
  __builtin_amdgcn_sched_barrier(0);
  __syncthreads();
  for (int k0 = 0; k0 < kend; k0 += 2 * kSK) {
    // tile k0 sits in stage 0; tile k0 + 32 goes from set 1 to stage 1, set 1 then takes tile k0 + 96
    tile(Stage0{}, Set1{}, min(k0 + 3 * kSK, klast));
    // tile k0 + 32 sits in stage 1; tile k0 + 64 goes from set 0 to stage 0, set 0 then takes tile k0 + 128
    tile(Stage1{}, Set0{}, min(k0 + 4 * kSK, klast));
  }

  // sum_ij A_ij T_ij of the tile in float64; accumulator r of a lane is row (r / 4) * 8 + (lane / 32) * 4 + r % 4,
  // column lane % 32 of its 32 x 32 tile; rows and columns beyond m x n hold zeros
  double s[kForms];
#pragma unroll
  for (int f = 0; f < kForms; ++f) {
    const uint16_t* P = f == 1 ? a.W : first;
    const int np_ = f == 1 ? NW : ND;
    s[f] = 0.0;
#pragma unroll
    for (int tm = 0; tm < 2; ++tm)
#pragma unroll
      for (int tn = 0; tn < 2; ++tn)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int i = wm * 64 + tm * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
          const int j = wn * 64 + tn * 32 + (lane & 31);
          const int64_t at = (int64_t)(i0 + i) * a.np + j0 + j;
          double v = (double)bf16_val(P[at]);
          for (int p = 1; p < np_; ++p) v += (double)bf16_val(P[p * planeA + at]);
          s[f] = fma((double)acc[f][tm][tn][r], v, s[f]);
        }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s[f] += __shfl_xor(s[f], off);
    if (lane == 0) red[f][wave] = s[f];
  }
  __syncthreads();
  if (tid == 0) {
    const int64_t tile = (int64_t)rt * gridDim.y + ct, tiles = (int64_t)gridDim.x * gridDim.y;
#pragma unroll
    for (int f = 0; f < kForms; ++f) {
      a.partial[(f == 1 || blockIdx.z ? tiles : 0) + tile] = (red[f][0] + red[f][1]) + (red[f][2] + red[f][3]);
    }
  }
}

// The same products in tiles of 256 x 128 for layers that have enough of them: eight waves, two per SIMD, 64 x 64 each.
// The pieces go from memory straight into LDS (buffer_load ... lds, inline assembly, waited for by count: the
// compiler would wait for all of them before each LDS read), two k-tiles of 32, rows of 64 bytes whose 16-byte slot s lies at
// s ^ (row / 4 % 4): the fragment reads of sixteen neighbouring lanes cover the 64 banks.  Step j: the first 16
// k of tile j | barrier | the others; at the barrier every wave has read tile j, whose place tile j + 2 takes, and tile
// j + 1 has landed.  What goes between the MFMAs is written down in order.  A workgroup of the 128 x 128 kernel has one wave per
// SIMD, which waits out the barrier, the first fragments and the LDS stores of each k-tile by itself.
// Bound: MFMA (five piece products of 11008 x 4096 in about 770 us: 1.2 PFLOP/s; the 128 x 128 kernel 1091).
template <int ND, int NW, int NH>
__global__ __launch_bounds__(512, 2) void quad_form_wide_kernel(SplitArgs a) {
  extern __shared__ __attribute__((aligned(16))) char wide_lds[];
  __shared__ double red[2][8];
  typedef __attribute__((address_space(3))) char lds_char;
  constexpr int NA = ND + NW, kRow = 64, kPieceA = kWideM * kRow, kPieceB = kT * kRow, kStage = NA * kPieceA + NH * kPieceB;
  constexpr int kRequestsA = NA * kWideM / 16, kRequests = kRequestsA + NH * kT / 16, kOwn = kRequests / 8;   // of 16 rows
  static_assert(kRequests % 8 == 0, "the same number for each wave");
  // Up to kSlab rows of tiles at a time, the widest column tiles first: the 256 workgroups in flight walk along k together
  // and read 16 strips of D and W and 16 of Hu (all rows of tiles at a time, 43 strips and 6: 1348 us for 11008 x 4096 instead of
  // 967).  Sixteen or eight rows put a strip on one XCD (workgroup ids = x mod 8) and its L2; fifteen do not:
  // 1262 us.  What is left over comes first, so that the narrow tiles of many rows are the last to start (2504 x 6971 with
  // its last two rows of tiles at the end: 894 us).
  const int rts = (a.mp + kWideM - 1) / kWideM, cts = a.np / kT;
  int row = 0, height = rts % 8 ? rts % 8 : (rts % kSlab ? rts % kSlab : kSlab), at = blockIdx.x;
  while (at >= height * cts) {
    at -= height * cts;
    row += height;
    height = (rts - row) % kSlab ? 8 : kSlab;
  }
  const int rt = row + at % height, ct = cts - 1 - at / height;
  const int i0 = rt * kWideM, j0 = ct * kT;
  const int ktiles = (j0 + kT) / kSK;   // beyond them Hu is zero; a multiple of four
  const int lane = threadIdx.x & 63, wave = (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int64_t planeA = (int64_t)a.mp * a.np, planeB = (int64_t)a.np * a.np;
  const uint16_t* first = NW == 0 && blockIdx.z ? a.W : a.D;

  // a wave's requests: 16 rows of a piece each; rows past mp deliver zeros
  const uint32_t lbase = (uint32_t)(uintptr_t)(lds_char*)wide_lds;
  const uint32_t voff = (uint32_t)((lane >> 2) * a.np * 2 + (((lane & 3) ^ (lane >> 4)) << 4));
  i32x4 src[kOwn];
  uint32_t dst[kOwn];
#pragma unroll
  for (int r = 0; r < kOwn; ++r) {
    const int q = wave * kOwn + r;
    const bool is_a = q < kRequestsA;
    const int p = is_a ? q / (kWideM / 16) : (q - kRequestsA) / (kT / 16);
    const int row = (is_a ? q % (kWideM / 16) : (q - kRequestsA) % (kT / 16)) * 16;
    const uint16_t* plane = is_a ? (p < ND ? first + p * planeA : a.W + (p - ND) * planeA) : a.HuT + p * planeB;
    const int at = is_a ? i0 + row : j0 + row;
    const bool there = !is_a || at < a.mp;
    src[r] = buffer_at(plane + (int64_t)(there ? at : 0) * a.np, there ? (int64_t)a.np * 32 : 0);
    dst[r] = (uint32_t)__builtin_amdgcn_readfirstlane(lbase + (is_a ? p * kPieceA : NA * kPieceA + p * kPieceB) + row * kRow);
  }
  auto request = [&](auto r_, auto stage_, int tile) {
    constexpr int r = decltype(r_)::value;
    request_to_lds<16>(src[r], voff, (uint32_t)min(tile, ktiles - 1) * (kSK * 2), dst[r] + decltype(stage_)::value * kStage);
  };

  f32x16 acc[1 + (NW > 0)][2][2];
#pragma unroll
  for (int f = 0; f < 1 + (NW > 0); ++f)
#pragma unroll
    for (int tm = 0; tm < 2; ++tm)
#pragma unroll
      for (int tn = 0; tn < 2; ++tn)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[f][tm][tn][r] = 0.f;

  // fragment of a 32-row strip: lane l holds row l % 32, k = 8 (l / 32) .. + 7 of the 16-wide k-step
  uint32_t at_a[2][2], at_b[2][2];   // [stage][k-step]
#pragma unroll
  for (int st = 0; st < 2; ++st)
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const uint32_t in_row = (uint32_t)((lane & 31) * kRow + (((2 * ks + (lane >> 5)) ^ ((lane >> 2) & 3)) << 4));
      at_a[st][ks] = st * kStage + wm * 64 * kRow + in_row;
      at_b[st][ks] = st * kStage + NA * kPieceA + wn * 64 * kRow + in_row;
      asm volatile("" : "+v"(at_a[st][ks]), "+v"(at_b[st][ks]));   // kept, not formed again before every read
    }
  constexpr int kReads = 2 * (NA + NH);
  bf16x8 fa[2][NA][2], fb[2][NH][2];   // [k-step][piece][strip]
  auto read = [&](auto stage_, auto ks_, auto index) {   // in the order of their first use: the last pieces of Hu and the first of D
    constexpr int ks = decltype(ks_)::value, st = decltype(stage_)::value, t = decltype(index)::value & 1, k = decltype(index)::value >> 1;
    if constexpr (k < NH) {
      constexpr int p = NH - 1 - k;
      fb[ks][p][t] = *(const __attribute__((address_space(3))) bf16x8*)((const lds_char*)wide_lds + (at_b[st][ks] + p * kPieceB + t * 32 * kRow));
    } else {
      constexpr int p = k - NH;
      fa[ks][p][t] = *(const __attribute__((address_space(3))) bf16x8*)((const lds_char*)wide_lds + (at_a[st][ks] + p * kPieceA + t * 32 * kRow));
    }
  };
  // piece pa of an operand with piece pb of Hu for pa + pb < NH, the smallest products first; MFMA I of a k-step
  constexpr int kFull = NH * (NH + 1) / 2, kProducts = kFull + (NW == 0 ? 0 : (NW == 1 ? NH : kFull)), kMfma = 4 * kProducts;
  static_assert(NW <= 1 && ND == NH, "");
  auto mfma = [&](auto ks_, auto index) {
    constexpr int ks = decltype(ks_)::value, I = decltype(index)::value;
    constexpr auto product = [](int want) constexpr {   // order, piece of A
      int n = 0;
      for (int order = NH - 1; order >= 0; --order)
        for (int p = 0; p < NA; ++p) {
          const int pa = p < ND ? p : p - ND, pb = order - pa;
          if (pb < 0 || pb >= NH) continue;
          if (n++ == want) return p * 16 + pb;
        }
      return -1;
    };
    constexpr int code = product(I / 4), p = code / 16, pb = code % 16, f = p >= ND ? 1 : 0, tm = I >> 1 & 1, tn = I & 1;
    static_assert(code >= 0, "");
    acc[f][tm][tn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[ks][p][tm], fb[ks][pb][tn], acc[f][tm][tn], 0, 0, 0);
  };
  using std::integral_constant;
  typedef integral_constant<int, 0> Zero;
  typedef integral_constant<int, 1> One;
  // per MFMA of a half at most one fragment read and, in the second half, one request
  static_assert(kReads <= kMfma && kOwn <= kMfma, "");
  auto step = [&](auto stage_, int tile) {
    constexpr int S = decltype(stage_)::value;
    typedef integral_constant<int, S ^ 1> Other;
    static_for<kMfma>([&](auto i_) {
      constexpr int i = decltype(i_)::value;
      mfma(Zero{}, i_);
      if constexpr (i < kReads) read(stage_, One{}, i_);
      __builtin_amdgcn_sched_barrier(0);
    });
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    wait_requests<0>();   // tile + 1, requested a step ago
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    static_for<kMfma>([&](auto i_) {
      constexpr int i = decltype(i_)::value;
      mfma(One{}, i_);
      if constexpr (i < kReads) read(Other{}, Zero{}, i_);
      if constexpr (i < kOwn) request(i_, stage_, tile + 2);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  static_for<kOwn>([&](auto r) { request(r, Zero{}, 0); });
  static_for<kOwn>([&](auto r) { request(r, One{}, 1); });
  wait_requests<kOwn>();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  static_for<kReads>([&](auto i) { read(Zero{}, Zero{}, i); });
  for (int tile = 0; tile < ktiles; tile += 2) {
    step(Zero{}, tile);
    step(One{}, tile + 1);
  }
  wait_requests<0>();   // nothing may still be landing in LDS when the workgroup ends

  // sum_ij A_ij T_ij of the tile in float64; accumulator r of a lane is row (r / 4) * 8 + (lane / 32) * 4 + r % 4,
  // column lane % 32 of its 32 x 32 tile; rows and columns beyond m x n hold zeros, rows beyond mp are not there
  double sums[1 + (NW > 0)];
#pragma unroll
  for (int f = 0; f < 1 + (NW > 0); ++f) {
    const uint16_t* P = f == 1 ? a.W : first;
    constexpr int kMost = ND;
    const int np_ = f == 1 ? NW : ND;
    sums[f] = 0.0;
    if (i0 + wm * 64 < a.mp) {
#pragma unroll
      for (int tm = 0; tm < 2; ++tm)
#pragma unroll
        for (int tn = 0; tn < 2; ++tn) {
          uint16_t v[16][kMost];
#pragma unroll
          for (int r = 0; r < 16; ++r)
#pragma unroll
            for (int p = 0; p < kMost; ++p) {
              const int i = wm * 64 + tm * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
              const int j = wn * 64 + tn * 32 + (lane & 31);
              v[r][p] = p < np_ ? P[p * planeA + (int64_t)(i0 + i) * a.np + j0 + j] : (uint16_t)0;
            }
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            double x = (double)bf16_val(v[r][0]);
#pragma unroll
            for (int p = 1; p < kMost; ++p) x += (double)bf16_val(v[r][p]);
            sums[f] = fma((double)acc[f][tm][tn][r], x, sums[f]);
          }
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sums[f] += __shfl_xor(sums[f], off);
    if (lane == 0) red[f][wave] = sums[f];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const int64_t tile = (int64_t)rt * cts + ct, tiles = (int64_t)rts * cts;
#pragma unroll
    for (int f = 0; f < 1 + (NW > 0); ++f) {
      double sum = 0.0;
#pragma unroll
      for (int w = 0; w < 8; ++w) sum += red[f][w];
      a.partial[(f == 1 || blockIdx.z ? tiles : 0) + tile] = sum;
    }
  }
}

__global__ __launch_bounds__(256) void finish_kernel(const double* __restrict__ partial, int tiles,
                                                     double* out) {
  __shared__ double red[2][256];
  for (int z = 0; z < 2; ++z) {
    double s = 0.0;
    for (int i = threadIdx.x; i < tiles; i += 256) s += partial[(int64_t)z * tiles + i];
    red[z][threadIdx.x] = s;
  }
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) {
      red[0][threadIdx.x] += red[0][threadIdx.x + w];
      red[1][threadIdx.x] += red[1][threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double num = red[0][0], den = red[1][0];
    out[0] = sqrt(num / den);
    out[1] = num;
    out[2] = den;
  }
}

}  // namespace

static size_t partial_bytes(int64_t m, int64_t n) {
  const size_t tiles = (size_t)ceil_div(m, Tile::BM) * (size_t)ceil_div(n, Tile::BN);
  return align_up(2 * tiles * sizeof(double), 256);
}

static size_t bytes_f64_form(int64_t m, int64_t n) {
  return partial_bytes(m, n) + align_up(2 * (size_t)m * (size_t)n * sizeof(double), 256);
}

static size_t partial_split_bytes(int64_t mp, int64_t np) {
  return align_up(2 * (size_t)(mp / kT) * (size_t)(np / kT) * sizeof(double), 256);
}

static size_t pieces_bytes(int64_t rows, int64_t cols) {
  return align_up(kMaxPieces * (size_t)rows * (size_t)cols * sizeof(uint16_t), 256);
}

static size_t bytes_split_form(int64_t m, int64_t n) {
  const int64_t mp = ceil_div(m, kT) * kT, np = ceil_div(n, kT) * kT;
  return partial_split_bytes(mp, np) + 2 * pieces_bytes(mp, np) + pieces_bytes(np, np);
}

// the caller asks before it says which storage type W has: enough for either form
size_t layer_error_workspace_bytes(int64_t m, int64_t n) {
  const size_t a = bytes_f64_form(m, n), b = bytes_split_form(m, n);
  return a > b ? a : b;
}

template <int ND, int NW, int NH>
static bool launch_wide(const SplitArgs& a, hipStream_t st) {
  constexpr int lds = 2 * ((ND + NW) * kWideM + NH * kT) * 64;
  if (!lds_opt_in<quad_form_wide_kernel<ND, NW, NH>>(lds)) return false;
  const dim3 g((unsigned)(ceil_div(a.mp, kWideM) * (a.np / kT)), 1, NW == 0 ? 2u : 1u);
  quad_form_wide_kernel<ND, NW, NH><<<g, 512, lds, st>>>(a);
  return true;
}

template <int ND, int NW, int NH>
static bool launch_split(const SplitArgs& a, hipStream_t st) {
  const int lds = 2 * (ND + NW + NH) * kT * kSP * (int)sizeof(uint16_t);
  if (!lds_opt_in<quad_form_split_kernel<ND, NW, NH>>(lds)) return false;
  const dim3 g((unsigned)(a.mp / kT), (unsigned)(a.np / kT), NW == 0 ? 2u : 1u);
  quad_form_split_kernel<ND, NW, NH><<<g, 256, lds, st>>>(a);
  return true;
}

static ptq_status launch_split_form(const void* W, ptq_dtype wdt, int64_t ldw, const double* Wq, int64_t m, int64_t n,
                                    const double* H, int64_t ldh, double* out, void* ws, hipStream_t st) {
  const int64_t mp = ceil_div(m, kT) * kT, np = ceil_div(n, kT) * kT;
  char* base = static_cast<char*>(ws);
  double* partial = reinterpret_cast<double*>(base);
  uint16_t* Dp = reinterpret_cast<uint16_t*>(base + partial_split_bytes(mp, np));
  uint16_t* Wp = reinterpret_cast<uint16_t*>(reinterpret_cast<char*>(Dp) + pieces_bytes(mp, np));
  uint16_t* HuT = reinterpret_cast<uint16_t*>(reinterpret_cast<char*>(Wp) + pieces_bytes(mp, np));
  const unsigned ga = (unsigned)ceil_div(mp * np / 4, 256);
  const dim3 gh((unsigned)(np / 32), (unsigned)(np / 32));
  int tiles = (int)((mp / kT) * (np / kT));
  SplitArgs a{Dp, Wp, HuT, (int)mp, (int)np, partial};
  // 256 x 128 tiles where there are enough for 256 workgroups to end together: the widest take 512 / tiles of the average
  // workgroup's time.  In bfloat16 from 448 on (whole call, 128 x 128 and 256 x 128 tiles: 2048 x 7168 626 and 596 us, 2304 x 7168
  // 698 and 638, 4096 x 4096 420 and 382, 11008 x 4096 1187 and 967; below, 2048 x 6144 (384) 487 and 560, 2304 x 6144 (432) 536
  // and 562, 2560 x 5120 (400) 422 and 426), from 384 where the rows of tiles are twelve or more, whose strips of D and W
  // neighbours share (3072 x 4096 325 and 315, 3328 x 4096 377 and 340, 5120 x 2560 228 and 209; 2560 x 4096 (320) 296 and 292,
  // 4096 x 2560 (320) 182 and 184).  In float32 both traces' tiles count: from 384 on (4096 x 11008 3548 and 3091, 1024 x 8192
  // 720 and 605, 640 x 8192 549 and 513, 3072 x 2048 136 and 132; 640 x 7168 (336) 392 and 420, 2048 x 2048 (256) 89 and 98; a loss
  // only near 6144 columns, 1408 to 2048 rows, 3 to 7 %).  Seven rows of tiles, whose strips go round the XCDs and are few, lose in
  // either type (1792 x 4096 in float32 272 and 299, 1792 x 11008 in bfloat16 1410 and 1504).
  const int64_t wide_rows = ceil_div(mp, kWideM), wide_tiles = wide_rows * (np / kT);
  const bool wide = m * n >= kTwoPiecesFrom && wide_rows != 7 &&
                    (wdt == PTQ_BF16 ? wide_tiles >= (wide_rows >= 12 ? 384 : 448) : 2 * wide_tiles >= 384);
  if (wide) tiles = (int)wide_tiles;
  auto run = [&](auto pieces) -> bool {
    constexpr int P = decltype(pieces)::value;
    if (wdt == PTQ_F32)
      split_weights_kernel<PTQ_F32, P><<<ga, 256, 0, st>>>(W, ldw, Wq, (int)m, (int)n, (int)mp, (int)np, Dp, Wp);
    else
      split_weights_kernel<PTQ_BF16, P><<<ga, 256, 0, st>>>(W, ldw, Wq, (int)m, (int)n, (int)mp, (int)np, Dp, Wp);
    split_hu_kernel<P><<<gh, 256, 0, st>>>(H, ldh, (int)n, (int)np, HuT);
    if constexpr (P == 2) {
      if (wide) return wdt == PTQ_BF16 ? launch_wide<P, 1, P>(a, st) : launch_wide<P, 0, P>(a, st);
    }
    if (wdt == PTQ_BF16) return launch_split<P, 1, P>(a, st);
    return launch_split<P, 0, P>(a, st);   // both traces in one launch (float32 512 x 512: 38.4 us for the call as two, now 24.8; 320 x 2856 148 and 87)
  };
  const bool ok = (m * n >= kTwoPiecesFrom) ? run(std::integral_constant<int, 2>{}) : run(std::integral_constant<int, 3>{});
  if (!ok) return PTQ_ERR_HIP;
  finish_kernel<<<1, 256, 0, st>>>(partial, tiles, out);
  PTQ_HIP_CHECK_LAUNCH();
  return PTQ_OK;
}

ptq_status layer_error_launch(const void* W, ptq_dtype wdt, int64_t ldw, const double* Wq, int64_t m,
                              int64_t n, const double* H, int64_t ldh, double* out, void* ws,
                              size_t ws_bytes, hipStream_t st) {
  if (ws_bytes < layer_error_workspace_bytes(m, n)) return PTQ_ERR_WORKSPACE;
  if (wdt == PTQ_F32 || wdt == PTQ_BF16) return launch_split_form(W, wdt, ldw, Wq, m, n, H, ldh, out, ws, st);
  if (wdt != PTQ_F64) return PTQ_ERR_DTYPE;
  double* partial = static_cast<double*>(ws);
  double* A2 = reinterpret_cast<double*>(static_cast<char*>(ws) + partial_bytes(m, n));
  const unsigned wg = (unsigned)ceil_div(m * n, 256);
  widen_kernel<<<wg, 256, 0, st>>>(static_cast<const double*>(W), ldw, Wq, (int)m, (int)n, A2);
  ErrArgs a{A2, (int)m, (int)n, H, ldh, partial};
  dim3 g(2 * (unsigned)ceil_div(m, Tile::BM), (unsigned)ceil_div(n, Tile::BN));
  const int tiles = (int)(g.x / 2 * g.y);
  constexpr int lds = Tile::kSmemDoubles * (int)sizeof(double);
  if (!lds_opt_in<quad_form_kernel>(lds)) return PTQ_ERR_HIP;
  quad_form_kernel<<<g, 256, lds, st>>>(a);
  finish_kernel<<<1, 256, 0, st>>>(partial, tiles, out);
  PTQ_HIP_CHECK_LAUNCH();
  return PTQ_OK;
}

}  // namespace ptq
