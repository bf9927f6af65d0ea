// Proxy-Hessian accumulation  H += X^T X  (upper triangle), X tokens x channels.
//
// bf16 path.  Tokens are the contraction index and the slow axis of X, while
// the matrix cores want, per lane, eight consecutive k for ONE channel.  The
// tile is therefore staged in LDS exactly as it lies in memory ([token][channel])
// and transposed on the way to registers: a lane reads the dword holding
// channels (2p, 2p+1) for eight tokens and two byte-permutes per pair of tokens
// split it into the fragment of channel 2p and the fragment of channel 2p+1.
// Even channels feed one 32x32x16 MFMA tile, odd channels the next one, so the
// output rows/columns of a wave are an interleaving of its two tiles.  Both
// operands are built the same way, hence any k order inside a fragment cancels.
//
// Products of two bf16 numbers are exact in float32.  A workgroup accumulates
// its 128 x 128 tile in float32 over at most 8192 tokens and stores that
// partial tile; a second kernel adds the partial tiles into H in float64 in a
// fixed order, so the result is bit-reproducible from run to run.  (Layers from 2048
// channels on: a 256 x 256-tile kernel, which adds to H by itself where the tokens
// are few enough for one split.)
//
// float32 activations: hessian_f32.hip (float64 matrix cores, 64 x 64 or 128 x 128 tiles), same
// partial scheme with float64 partial tiles.
#include "common.h"
#include "lds_dma.h"

namespace ptq {
namespace {

constexpr int kTile = 128;      // bf16 macro tile (channels x channels)
constexpr int kKT = 32;         // tokens per LDS stage
constexpr int kPitch = kTile + 8;  // bf16 elements; 272-byte rows
constexpr int kMaxChunk = 8192;      // tokens summed in float32 before the float64 reduction
constexpr int kMaxChunkBig = 20480;  // ... in the 256 x 256-tile kernel (fewer, larger partial tiles)
constexpr int kMaxChunkHuge = 65536; // ... and once a split alone fills the chip several times over

constexpr int kTile32 = 64;          // float32 activations: tile of narrow layers
constexpr int kTile32Wide = 128;     // ... and from kWide32From channels on
constexpr int64_t kWide32From = 1024;
constexpr int kKT32 = 16;

__device__ __forceinline__ void tile_from_linear(int lin, int ntb, int& I, int& J) {
  // upper-triangular tile list, row by row: row I holds ntb - I tiles
  int i = 0;
  while (lin >= ntb - i) {
    lin -= ntb - i;
    ++i;
  }
  I = i;
  J = i + lin;
}

__global__ __launch_bounds__(256) void hessian_bf16_kernel(const uint16_t* __restrict__ X, int64_t ldx,
                                                           int64_t t, int n, int64_t tok0, int chunk,
                                                           int ntb, float* __restrict__ partial) {
  __shared__ __attribute__((aligned(16))) uint16_t As[kKT * kPitch];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[kKT * kPitch];
  int I, J;
  tile_from_linear(blockIdx.x, ntb, I, J);
  const bool diag = (I == J);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wi = wave >> 1, wj = wave & 1;
  const int64_t kbeg = tok0 + (int64_t)blockIdx.y * chunk;
  const int64_t kend = (kbeg + chunk < t) ? kbeg + chunk : t;

  // global -> LDS map: 16 threads cover one token row (8 channels = 16 bytes each)
  const int lrow = tid >> 4, lcol = (tid & 15) * 8;
  const bool a_in = (I * kTile + lcol) < n, b_in = (J * kTile + lcol) < n;
  const uint16_t* ga = X + I * kTile + lcol;
  const uint16_t* gb = X + J * kTile + lcol;

  f32x16 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;

  uint4 ra[2], rb[2];
  auto fetch = [&](int64_t k0) {
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const int64_t k = k0 + lrow + 16 * p;
      const bool kin = k < kend;
      ra[p] = (kin && a_in) ? *reinterpret_cast<const uint4*>(ga + k * ldx) : uint4{0, 0, 0, 0};
      if (!diag) rb[p] = (kin && b_in) ? *reinterpret_cast<const uint4*>(gb + k * ldx) : uint4{0, 0, 0, 0};
    }
  };
  auto stash = [&]() {
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      *reinterpret_cast<uint4*>(&As[(lrow + 16 * p) * kPitch + lcol]) = ra[p];
      if (!diag) *reinterpret_cast<uint4*>(&Bs[(lrow + 16 * p) * kPitch + lcol]) = rb[p];
    }
  };
  // fragments of the even and the odd channels of a 64-channel strip
  auto fragments = [&](const uint16_t* T, int strip, int ks, bf16x8 (&f)[2]) {
    const int p = lane & 31, kg = lane >> 5;
    uint32_t d[8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
      d[i] = *reinterpret_cast<const uint32_t*>(&T[(ks * 16 + kg * 8 + i) * kPitch + strip * 64 + 2 * p]);
    uint32_t ev[4], od[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      ev[i] = __builtin_amdgcn_perm(d[2 * i + 1], d[2 * i], 0x05040100u);
      od[i] = __builtin_amdgcn_perm(d[2 * i + 1], d[2 * i], 0x07060302u);
    }
    typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
    f[0] = __builtin_bit_cast(bf16x8, u32x4{ev[0], ev[1], ev[2], ev[3]});
    f[1] = __builtin_bit_cast(bf16x8, u32x4{od[0], od[1], od[2], od[3]});
  };

  if (kbeg < kend) {
    fetch(kbeg);
    for (int64_t k0 = kbeg; k0 < kend; k0 += kKT) {
      __syncthreads();
      stash();
      __syncthreads();
      if (k0 + kKT < kend) fetch(k0 + kKT);
      const uint16_t* Bt = diag ? As : Bs;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        bf16x8 fa[2], fb[2];
        fragments(As, wi, ks, fa);
        fragments(Bt, wj, ks, fb);
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int b = 0; b < 2; ++b)
            acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[a], fb[b], acc[a][b], 0, 0, 0);
      }
    }
  }

  float* out = partial + ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * (kTile * kTile);
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int il = (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
        const int jl = lane & 31;
        out[(wi * 64 + 2 * il + a) * kTile + wj * 64 + 2 * jl + b] = acc[a][b][r];
      }
}

// ---- large layers: 256 x 256 tile, each wave 128 x 128 (4 x 4 MFMA tiles) ------
// The tile's operands go from global memory straight into LDS (buffer_load ... lds,
// 16 bytes per lane, no staging registers) as they lie in memory, [token][channel], into
// a ring of four 32-token stages.  The transposition to "eight consecutive tokens of one
// channel per lane" is done by the LDS itself: ds_read_b64_tr_b16 hands a lane four tokens
// of its channel, two such reads make one MFMA operand.  Per 16 tokens a wave issues 16
// of these reads and 16 MFMAs (32 cycles each), accumulators fill the 256 AGPRs.
//
// LDS layout of a stage: A part (32 token rows x 512 bytes) then B part.  A row holds 32
// chunks of 16 bytes (8 channels); chunk c of token row r sits at position c ^ swz(r & 3),
// which spreads the 16 chunks a half-wave reads (four token rows x 64 bytes) over all
// banks.  A DMA instruction writes 64 consecutive chunks (two token rows) in lane order, so
// the swizzle is applied on the global side: lane j of the instruction fetches the chunk
// that belongs at position j & 31.
//
// Tokens past the end of the chunk are never fetched: the buffer descriptor ends with the
// chunk and out-of-range lanes deliver zeros.  Channels past n (last tile row / column
// only) fetch some valid channel instead; the outputs they feed lie outside the matrix and
// are dropped by the reduction.
//
// The DMA requests are those of lds_dma.h.
constexpr int kBT = 256;
constexpr int kBKS = 32;                          // tokens per stage
constexpr int kBRing = 4;                         // stages in LDS
constexpr int kBRow = kBT * 2;                    // bytes per token row of the A part
constexpr int kBPart = kBKS * kBRow;              // A part: 16 KB
constexpr size_t kBigLdsBytes = (size_t)kBRing * 2 * kBPart;  // 128 KB

typedef __attribute__((__vector_size__(4 * sizeof(short)))) short i16x4;

__device__ __forceinline__ int swz(int row) { return ((row & 1) * 10) | ((row & 2) * 2); }

// rows of MFMA tiles that a wave of big_tile has in this role
template <int ROLE>
constexpr int role_rows = ROLE == 2 ? 2 : (ROLE == 3 ? 0 : 4);

// A wave's tile is 128 x 32 NB: NB = 4, the 256 x 256 tile; NB = 2, one half (`half_tile`, 128 columns) of an
// off-diagonal 256 x 256 tile, with a B part of half the size.  On a diagonal tile both operands come from the A part;
// waves 0 and 3 take its two diagonal quadrants (ten of sixteen MFMA tiles) and wave 1 the off-diagonal one, which
// keeps the workgroup in step with those of whole tiles beside it (they share their operands in the L2); SHARED: waves 1
// and 2 take half of it each, for half tiles and for short splits (kSharedTokens).
template <bool diag, int NB, bool SHARED, bool DIRECT>
__device__ __forceinline__ void big_tile(const uint16_t* __restrict__ X, int64_t ldx, int64_t t, int n,
                                         int64_t tok0, int chunk, int I, int J, int half_tile, int split,
                                         float* __restrict__ out, double* __restrict__ H, int64_t ldh, uint16_t* hs) {
  static_assert(NB == 4 || (NB == 2 && !diag), "");
  constexpr int kBRowB = 128 * NB;                  // bytes per token row of the B part
  constexpr int kBStage = kBPart + kBKS * kBRowB;   // 32 or 24 KB
  typedef __attribute__((address_space(3))) char lds_char;
  typedef __attribute__((address_space(3))) i16x4 lds_i16x4;
  lds_char* lds = (lds_char*)hs;
  const uint32_t lbase = (uint32_t)(uintptr_t)lds;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // rows 128 wi + 64 * low .., columns 32 NB wj of the tile (low: the second half of a shared quadrant)
  const int wi = SHARED ? wave == 3 : wave >> 1, wj = SHARED ? wave != 0 : wave & 1;
  const int low = SHARED && wave == 2;
  const int64_t kbeg = tok0 + (int64_t)split * chunk;
  const int64_t kend = (kbeg + chunk < t) ? kbeg + chunk : t;
  const int64_t len = kend - kbeg;

  f32x16 acc[4][NB];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;

  if (len > 0) {
    const int nstage = (int)((len + kBKS - 1) / kBKS);
    constexpr int L = diag ? 4 : 4 + NB;  // DMA instructions per stage and wave

    // descriptor over the chunk's tokens (uniform, kept in scalar registers)
    i32x4 rs = buffer_at(X + kbeg * ldx, len * ldx * 2);   // bytes, < 2^32 (host)
    const uint32_t stage_step = __builtin_amdgcn_readfirstlane((uint32_t)(kBKS * ldx * 2));

    // per-lane byte offsets of the DMA instructions of a part, inside a stage (the descriptor advances): one brings
    // two token rows of 32 chunks, or four of 16
    uint32_t voA[4], voB[NB];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = 8 * i + 2 * wave + (lane >> 5);
      int col = I * kBT + 8 * ((lane & 31) ^ swz(row));
      if (col >= n) col = I * kBT;
      voA[i] = (uint32_t)((row * ldx + col) * 2);
    }
    const int col0 = J * kBT + (NB == 2 ? 128 * half_tile : 0);
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      constexpr int kPerRow = 8 * NB;   // chunks
      const int row = (32 / NB) * i + (8 / NB) * wave + lane / kPerRow;
      int col = col0 + 8 * ((lane % kPerRow) ^ swz(row));
      if (col >= n) col = J * kBT;
      voB[i] = (uint32_t)((row * ldx + col) * 2);
    }
    // per-lane LDS read addresses inside a stage, one per MFMA tile of the wave's strips
    uint32_t adA[4], adB[NB];
    {
      const int g = lane >> 4, h = g & 1, kg = g >> 1, j = lane & 15, r = j >> 2, q = j & 3;
      const int row = kg * 8 + r;
#pragma unroll
      for (int T = 0; T < 4; ++T) {
        const int c = wi * 16 + low * 8 + (T & (low ? 1 : 3)) * 4 + 2 * h + (q >> 1);
        adA[T] = row * kBRow + ((c ^ swz(r)) * 16) + (q & 1) * 8;
      }
#pragma unroll
      for (int T = 0; T < NB; ++T) {
        const int c = wj * 4 * NB + T * 4 + 2 * h + (q >> 1);
        adB[T] = (diag ? 0 : kBPart) + row * kBRowB + ((c ^ swz(r)) * 16) + (q & 1) * 8;
      }
    }
    // fragment of eight tokens: rows +0..3 and +4..7 relative to the lane's row (of `pitch` bytes)
    auto read_one = [&](uint32_t addr, int pitch) -> bf16x8 {
      const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(lds + addr));
      const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(lds + addr + 4 * pitch));
      return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    // DMA instruction q of a stage (A rows first, then B rows) into the slot at dst
    auto dma_q = [&](int q, uint32_t dst) {
      if (q < 4) request_to_lds(rs, voA[q], dst + q * 4096);
      else request_to_lds(rs, voB[q - 4], dst + kBPart + (q - 4) * 4096);
    };
    // One stage on: the descriptor moves (base up, extent down, never below zero -- past the end of the chunk every
    // lane is out of range and delivers zeros), the per-lane offsets stay.  Scalar work, where advancing the
    // eight per-lane offsets costs the wave eight vector instructions per stage.
    auto dma_advance = [&]() {
      const uint64_t base = (((uint64_t)(uint32_t)rs[1] << 32) | (uint32_t)rs[0]) + stage_step;
      uint32_t left;
      // (the compiler would form the saturating difference in a vector register, and a request has to wait five states
      // for a descriptor that comes out of one)
      asm("s_sub_u32 %0, %1, %2\n\ts_cselect_b32 %0, 0, %0" : "=s"(left) : "s"(rs[2]), "s"(stage_step) : "scc");
      rs[0] = (int)__builtin_amdgcn_readfirstlane((uint32_t)base);
      rs[1] = (int)__builtin_amdgcn_readfirstlane((uint32_t)(base >> 32));
      rs[2] = (int)left;
    };
    // The MFMAs of 16 tokens on (fa, fb) while the next fragments (na, nb) are read, `soA` / `soB` bytes on.  L/2 DMA
    // instructions, q0 onwards, go between the four groups of MFMAs: issued in one burst they fill the
    // memory pipeline's queue and the wave (hence its MFMAs) stalls.
    // ROLE: 0 = all MFMA tiles of the wave; on a diagonal tile 1 = only those on or above the diagonal (the quadrant is
    // itself a diagonal block of H), 2 = the upper two rows of them (a shared quadrant), 3 = none (the quadrant lies below
    // the diagonal; the wave only moves data).
    auto group_order = [&](auto role, auto g_) {   // what is asked of the scheduler for group g
      constexpr int ROLE = decltype(role)::value, g = decltype(g_)::value;
      constexpr int M = ROLE == 1 ? 4 - g : NB;
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);  // DS read
      if constexpr (M > 1) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if constexpr (g < NB) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
      if constexpr (M > 2) __builtin_amdgcn_sched_group_barrier(0x008, M - 2, 0);
    };
    // the request that goes after group g of a half: q0 + this, or -1
    auto request_after = [](int g) constexpr { return L == 8 ? g : (L == 6 ? (g < 3 ? g : -1) : (g & 1 ? g >> 1 : -1)); };
    auto half = [&](auto role, const bf16x8 (&fa)[4], const bf16x8 (&fb)[NB], bf16x8 (&na)[4], bf16x8 (&nb)[NB],
                    uint32_t soA, uint32_t soB, int q0, uint32_t dst) {
      constexpr int ROLE = decltype(role)::value;
      static_for<4>([&](auto g_) {
        constexpr int g = decltype(g_)::value;
        if constexpr (g < role_rows<ROLE>) na[g] = read_one(soA + adA[g], kBRow);
        if constexpr (g < NB && ROLE != 3) nb[g] = read_one(soB + adB[g], kBRowB);
        if constexpr (g < role_rows<ROLE>) {
#pragma unroll
          for (int b = (ROLE == 1 ? g : 0); b < NB; ++b)
            acc[g][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[g], fb[b], acc[g][b], 0, 0, 0);
          group_order(role, g_);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (request_after(g) >= 0) dma_q(q0 + request_after(g), dst);
        __builtin_amdgcn_sched_barrier(0);
      });
    };

    // prologue: stages 0, 1, 2 and the first half of stage 3 are requested; stage 0 must have
    // landed.  Stages past the end of the chunk are requested like the others and deliver zeros.
#pragma unroll
    for (int s = 0; s < kBRing - 1; ++s) {
#pragma unroll
      for (int q = 0; q < L; ++q) dma_q(q, lbase + s * kBStage + wave * 1024);
      dma_advance();
    }
#pragma unroll
    for (int q = 0; q < L / 2; ++q) dma_q(q, lbase + (kBRing - 1) * kBStage + wave * 1024);
    wait_requests<2 * L + L / 2>();
    __builtin_amdgcn_s_barrier();

    // Iteration s: tokens 0..15 of stage s | barrier | tokens 16..31.  At the barrier every wave
    // has finished reading stage s, so its slot is refilled with stage s + 4: the first half of
    // those DMA instructions is spread over the second half of iteration s, the rest over the
    // first half of iteration s + 1.  In issue order the requests outstanding at the barrier are
    // those of stages s+1, s+2, s+3, and stage s+1 is the one that must have landed.
    // The same half with the ring slot known at compile time: SO (LDS offset of the tokens to read) folds into the
    // immediate offset of the LDS reads -- from a second set of per-lane addresses, 64 KB further on, for the upper
    // two slots, since the immediate has 16 bits -- and DST (slot being refilled) into the immediate of the request's
    // scalar add.  With a run-time slot every pair of reads and every request needs an add of its own, and this
    // loop is bound by what a wave issues besides its MFMAs.
    uint32_t hiA[4], hiB[NB];
#pragma unroll
    for (int T = 0; T < 4; ++T) {
      hiA[T] = adA[T] + 65536u;
      // (opaque to the compiler, or it forms them again before every use instead of keeping the registers)
      asm volatile("" : "+v"(hiA[T]));
    }
#pragma unroll
    for (int T = 0; T < NB; ++T) {
      hiB[T] = adB[T] + 65536u;
      asm volatile("" : "+v"(hiB[T]));
    }
    const uint32_t wbase = lbase + wave * 1024;
    auto half_at = [&](auto role, auto slot_, auto second_, auto q0_, auto dst_, const bf16x8 (&fa)[4], const bf16x8 (&fb)[NB],
                       bf16x8 (&na)[4], bf16x8 (&nb)[NB]) {
      constexpr int ROLE = decltype(role)::value;
      constexpr uint32_t SA = decltype(slot_)::value + (decltype(second_)::value ? 16 * kBRow : 0), DST = decltype(dst_)::value;
      constexpr uint32_t SB = decltype(slot_)::value + (decltype(second_)::value ? 16 * kBRowB : 0);
      constexpr int Q0 = decltype(q0_)::value;
      constexpr bool HIA = SA >= 65536u, HIB = SB >= 65536u;
      constexpr uint32_t soA = HIA ? SA - 65536u : SA, soB = HIB ? SB - 65536u : SB;
      static_for<4>([&](auto g_) {
        constexpr int g = decltype(g_)::value;
        if constexpr (g < role_rows<ROLE>) na[g] = read_one(soA + (HIA ? hiA[g] : adA[g]), kBRow);
        if constexpr (g < NB && ROLE != 3) nb[g] = read_one(soB + (HIB ? hiB[g] : adB[g]), kBRowB);
        if constexpr (g < role_rows<ROLE>) {
#pragma unroll
          for (int b = (ROLE == 1 ? g : 0); b < NB; ++b)
            acc[g][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[g], fb[b], acc[g][b], 0, 0, 0);
          group_order(role, g_);
        }
        __builtin_amdgcn_sched_barrier(0);
        constexpr int at = L == 8 ? g : (L == 6 ? (g < 3 ? g : -1) : (g & 1 ? g >> 1 : -1));
        if constexpr (at >= 0) {
          constexpr int q = Q0 + at;
          if constexpr (q < 4) request_to_lds_at<DST + q * 4096>(rs, voA[q], wbase);
          else request_to_lds_at<DST + kBPart + (q - 4) * 4096>(rs, voB[q - 4], wbase);
        }
        __builtin_amdgcn_sched_barrier(0);
      });
    };

    // Iteration s: tokens 0..15 of stage s | barrier | tokens 16..31.  At the barrier every wave
    // has finished reading stage s, so its slot is refilled with stage s + 4: the first half of
    // those DMA instructions is spread over the second half of iteration s, the rest over the
    // first half of iteration s + 1.  In issue order the requests outstanding at the barrier are
    // those of stages s+1, s+2, s+3, and stage s+1 is the one that must have landed.
    // Four iterations per trip of the loop, one per ring slot; what is left over (the number of stages
    // is not a multiple of four) takes the form with a run-time slot.
    auto main_loop = [&](auto role) {
      constexpr int ROLE = decltype(role)::value;
      using std::integral_constant;
      bf16x8 fa0[4], fb0[NB], fa1[4], fb1[NB];
#pragma unroll
      for (int T = 0; T < role_rows<ROLE>; ++T) fa0[T] = read_one(adA[T], kBRow);
#pragma unroll
      for (int T = 0; T < (ROLE == 3 ? 0 : NB); ++T) fb0[T] = read_one(adB[T], kBRowB);
      auto iteration_at = [&](auto slot_) {
        constexpr uint32_t SLOT = decltype(slot_)::value;
        constexpr uint32_t slot_off = SLOT * kBStage, pend_off = ((SLOT + kBRing - 1) & (kBRing - 1)) * kBStage,
                           next_off = ((SLOT + 1) & (kBRing - 1)) * kBStage;
        half_at(role, integral_constant<uint32_t, slot_off>{}, std::true_type{}, integral_constant<int, L / 2>{},
                integral_constant<uint32_t, pend_off>{}, fa0, fb0, fa1, fb1);
        dma_advance();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        wait_requests<2 * L>();
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        half_at(role, integral_constant<uint32_t, next_off>{}, std::false_type{}, integral_constant<int, 0>{},
                integral_constant<uint32_t, slot_off>{}, fa1, fb1, fa0, fb0);
      };
      int s = 0;
      for (; s + kBRing <= nstage; s += kBRing) {
        iteration_at(integral_constant<uint32_t, 0>{});
        iteration_at(integral_constant<uint32_t, 1>{});
        iteration_at(integral_constant<uint32_t, 2>{});
        iteration_at(integral_constant<uint32_t, 3>{});
      }
      for (; s < nstage; ++s) {
        const uint32_t slot_off = (s & (kBRing - 1)) * kBStage;
        const uint32_t pend_off = ((s + kBRing - 1) & (kBRing - 1)) * kBStage;
        const uint32_t next_off = ((s + 1) & (kBRing - 1)) * kBStage;
        half(role, fa0, fb0, fa1, fb1, slot_off + 16 * kBRow, slot_off + 16 * kBRowB, L / 2, lbase + pend_off + wave * 1024);
        dma_advance();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        wait_requests<2 * L>();
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        half(role, fa1, fb1, fa0, fb0, next_off, next_off, 0, lbase + slot_off + wave * 1024);
      }
    };
    if constexpr (!diag) {
      main_loop(std::integral_constant<int, 0>{});
    } else if constexpr (SHARED) {
      if (wave == 1 || wave == 2) main_loop(std::integral_constant<int, 2>{});
      else main_loop(std::integral_constant<int, 1>{});
    } else {
      if (wave == 1) main_loop(std::integral_constant<int, 0>{});
      else if (wave == 2) main_loop(std::integral_constant<int, 3>{});
      else main_loop(std::integral_constant<int, 1>{});
    }
    wait_requests<0>();  // nothing may still be landing in LDS when the workgroup ends
  }

  // register r of MFMA tile (a, b): row 8 (r / 4) + 4 (lane / 32) + r % 4, column lane % 32
  const int il0 = wi * 128 + low * 64 + (lane >> 5) * 4, jl0 = (NB == 2 ? 128 * half_tile : 0) + wj * 32 * NB + (lane & 31);
  const int rows = SHARED && (wave == 1 || wave == 2) ? 2 : 4;   // MFMA tile rows of this wave
  if constexpr (DIRECT) {
    // The only split: straight into H, 16 entries of a lane at a time (8 or 4 rows of an MFMA tile across all of the wave's
    // columns) while the next 16 are on their way; entries outside the matrix or below the diagonal are loaded from some valid
    // place and not stored (a load under a condition would wait for the one before).  With each 16 waiting for their own
    // loads a workgroup pays the way to memory 8 or 16 times: calls of 2048 tokens n = 4096 54 -> 51 us, n = 8192 224 -> 182,
    // n = 11008 405 -> 350.  32 entries at a time spill.
    constexpr int kRows = 16 / NB, kSteps = 64 / kRows;
    double v[2][kRows][NB];
    auto load = [&](auto step) {
      constexpr int S = decltype(step)::value, a = S * kRows / 16, r0 = S * kRows % 16;
#pragma unroll
      for (int r = 0; r < kRows; ++r)
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          const int i = I * kBT + il0 + 32 * a + ((r0 + r) >> 2) * 8 + (r & 3), j = J * kBT + jl0 + 32 * b;
          v[S & 1][r][b] = H[(int64_t)min(i, n - 1) * ldh + min(j, n - 1)];
        }
    };
    load(std::integral_constant<int, 0>{});
    static_for<kSteps>([&](auto step) {
      constexpr int S = decltype(step)::value, a = S * kRows / 16, r0 = S * kRows % 16;
      if (a >= rows) return;
      if constexpr (S + 1 < kSteps) load(std::integral_constant<int, S + 1>{});
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = 0; r < kRows; ++r)
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          const int i = I * kBT + il0 + 32 * a + ((r0 + r) >> 2) * 8 + (r & 3), j = J * kBT + jl0 + 32 * b;
          if (j < n && i <= j) H[(int64_t)i * ldh + j] = v[S & 1][r][b] + (double)acc[a][b][r0 + r];
        }
      __builtin_amdgcn_sched_barrier(0);
    });
    return;
  }
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    if (a >= rows) break;
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int il = il0 + 32 * a + (r >> 2) * 8 + (r & 3);
        out[il * kBT + jl0 + 32 * b] = acc[a][b][r];
      }
  }
}

// Work order.  Workgroups are handed to the eight XCDs (each with its own L2) round-robin by
// workgroup id.  All (split, tile) items are laid out in one locality order -- split by split,
// and inside a split by super-tiles of 8 x 8 tiles.  The 256 workgroups in flight take 256
// consecutive items, and of those XCD x (ids = x mod 8) takes 32 consecutive ones: its L2 then
// serves a few channel strips over the same tokens, and the memory-side cache serves what the
// XCDs share (the same one or two splits, at most two slabs of tokens x n).
constexpr int kSuper = 8;

__device__ __forceinline__ void tile_in_locality_order(int r, int ntb, int& I, int& J) {
  const int ns = (ntb + kSuper - 1) / kSuper;
  for (int a = 0; a < ns; ++a) {
    const int ha = min(kSuper, ntb - a * kSuper);
    for (int b = a; b < ns; ++b) {
      const int hb = min(kSuper, ntb - b * kSuper);
      const int cnt = (a == b) ? ha * (ha + 1) / 2 : ha * hb;
      if (r < cnt) {
        int i, j;
        if (a == b) {
          i = 0;
          while (r >= ha - i) {
            r -= ha - i;
            ++i;
          }
          j = i + r;
        } else {
          i = r / hb;
          j = r - i * hb;
        }
        I = a * kSuper + i;
        J = b * kSuper + j;
        return;
      }
      r -= cnt;
    }
  }
  I = J = 0;  // not reached
}

// HALVES: an item is half of an off-diagonal tile (and the whole of a diagonal one: those come first, they take a
// quarter longer).  For calibration that arrives a few sequences at a time, where the tiles of a call alone do not
// fill the chip: n = 4096 has 136 tiles, but 256 such items.  Half a tile takes about 66 % of a whole one's time (three
// quarters of its operands pass through the LDS for half the MFMAs), so the split into halves is taken where it
// saves rounds of 256 workgroups.
// DIRECT: one split, added to H without a partial tile.  Bound: H's float64 update, 16 bytes per entry.
// Call of 2048 tokens, partial tiles and whole tiles before: n = 4096 90.1 -> 51 us, n = 5376 111 -> 83,
// n = 8192 325 -> 182, n = 11008 564 -> 350; n = 2048, seven splits either way, 40.0 and 40.7.
template <bool HALVES, bool SHARED, bool DIRECT>
__global__ __launch_bounds__(256) void hessian_bf16_big_kernel(const uint16_t* __restrict__ X, int64_t ldx,
                                                               int64_t t, int n, int64_t tok0, int chunk,
                                                               int ntb, int ntiles, int nsplits,
                                                               float* __restrict__ partial, double* __restrict__ H,
                                                               int64_t ldh) {
  extern __shared__ __attribute__((aligned(16))) uint16_t hs[];
  const int items = HALVES ? ntb * ntb : ntiles;
  const int total = items * nsplits;
  const int q = 256 * (blockIdx.x >> 8) + 32 * (blockIdx.x & 7) + ((blockIdx.x & 255) >> 3);
  if (q >= total) return;
  const int split = q / items;
  int k = q - split * items, I, J, half_tile = 0;
  if constexpr (HALVES) {
    if (k < ntb) {
      I = J = k;
    } else {   // the two halves of a tile above the diagonal, row by row of tiles
      k -= ntb;
      half_tile = k & 1;
      k >>= 1;
      I = 0;
      while (k >= ntb - 1 - I) {
        k -= ntb - 1 - I;
        ++I;
      }
      J = I + 1 + k;
    }
  } else {
    tile_in_locality_order(k, ntb, I, J);
  }
  const int lin = I * ntb - I * (I - 1) / 2 + (J - I);  // index in the row-major upper-triangular tile list
  float* out = partial + ((int64_t)split * ntiles + lin) * (kBT * kBT);
  if (I == J)
    big_tile<true, 4, SHARED, DIRECT>(X, ldx, t, n, tok0, chunk, I, J, 0, split, out, H, ldh, hs);
  else
    big_tile<false, HALVES ? 2 : 4, false, DIRECT>(X, ldx, t, n, tok0, chunk, I, J, half_tile, split, out, H, ldh, hs);
}

// H[upper] += sum over splits of the partial tiles, in float64, fixed order.  Four consecutive
// elements of a tile row per thread (TILE is a multiple of 4, so they share the row).
template <class PT, int TILE>
__global__ __launch_bounds__(256) void hessian_reduce_kernel(const PT* __restrict__ partial, int splits,
                                                             int ntiles, int ntb, int n,
                                                             double* __restrict__ H, int64_t ldh) {
  int I, J;
  tile_from_linear(blockIdx.x, ntb, I, J);
  const int e = (blockIdx.y * 256 + threadIdx.x) * 4;
  const int r = e / TILE, c = e % TILE;
  const int gi = I * TILE + r, gj = J * TILE + c;
  if (gi >= n || gj >= n || gi > gj + 3) return;
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  for (int sp = 0; sp < splits; ++sp) {
    const PT* src = partial + ((int64_t)sp * ntiles + blockIdx.x) * (TILE * TILE) + e;
    PT v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = src[q];
#pragma unroll
    for (int q = 0; q < 4; ++q) s[q] += (double)v[q];
  }
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (gj + q < n && gi <= gj + q) H[(int64_t)gi * ldh + gj + q] += s[q];
}

struct Plan {
  int tile, ntb, ntiles, chunk, splits_total, splits_launch;
  bool halves;   // 256-tile kernel: items of half a tile
  size_t tile_bytes;
};

constexpr int64_t kHalfCost = 66;   // percent of a whole tile's time that half a tile takes (measured with full rounds)
// Tokens of a split up to which whole tiles added to H share the off-diagonal quadrant of a diagonal tile: a short split ends
// with the update of H, which such a workgroup then starts earlier; in a long one the workgroups should keep in step.
// Shared and not: n = 16384 with 2048 tokens 862 and 883 us, 4096 1237 and 1267; n = 11008 with 2048 402 and 405, 4096
// 580 and 586, 16384 1675 and 1677, 20480 2047 and 2034, 46016 4428 and 4392; n = 9728 with 65536 4904 and 4865; n = 5632
// with 2048 to 20480 the same.  (Partial tiles are never shared: 262144 tokens x 11008 took 25.2 ms instead of 24.5.)
constexpr int kSharedTokens = 16384;
constexpr int64_t kBigFrom = 2048;                   // layers at least this wide use the 256-tile kernel
constexpr size_t kMaxPartialBytes = (size_t)1 << 30;  // partial tiles in flight per launch

// The 256-tile kernel addresses a chunk of tokens (and the ring's read-ahead past it) with
// 32-bit byte offsets, which bounds the row pitch.
bool big_kernel_fits(int64_t ldx) {
  return (kMaxChunkHuge + (kBRing + 1) * kBKS) * ldx * 2 < ((int64_t)1 << 32);
}

Plan make_plan(int64_t n, int64_t t, ptq_dtype dt, bool allow_big) {
  Plan p;
  const bool big = allow_big && (dt == PTQ_BF16) && n >= kBigFrom;
  p.tile = (dt == PTQ_BF16) ? (big ? kBT : kTile) : (n >= kWide32From ? kTile32Wide : kTile32);
  const int kt = (dt == PTQ_BF16) ? kKT : kKT32;
  p.ntb = (int)ceil_div(n, p.tile);
  p.ntiles = p.ntb * (p.ntb + 1) / 2;
  // Split the tokens so that the workgroups fill 256 CUs in whole rounds, with at most
  // max_chunk tokens summed in float32 by one workgroup: pick the split count with the
  // least (rounds x work per split).
  // (with >= 512 tiles the rounds are full for any split count, so longer float32 sums buy fewer partial tiles)
  const int64_t max_chunk = big ? (p.ntiles >= 512 ? kMaxChunkHuge : kMaxChunkBig) : kMaxChunk;
  const int64_t s_min = ceil_div(t > 0 ? t : 1, max_chunk);
  int64_t best_s = s_min, best_cost = -1;
  for (int64_t sp = s_min; sp < s_min + 64; ++sp) {
    int64_t ch = ceil_div(ceil_div(t > 0 ? t : 1, sp), kt) * kt;
    if (ch < 256 && sp > s_min) break;
    // + 1024: writing and re-reading a partial tile costs about as much as 1024 tokens
    const int64_t cost = ceil_div(p.ntiles * sp, 256) * (ch + 1024);
    if (best_cost < 0 || cost < best_cost) {
      best_cost = cost;
      best_s = sp;
    }
  }
  int64_t chunk = ceil_div(ceil_div(t > 0 ? t : 1, best_s), kt) * kt;
  if (chunk < kt) chunk = kt;
  p.chunk = (int)chunk;
  p.splits_total = (int)ceil_div(t > 0 ? t : 1, chunk);
  // Whole tiles alone decide how many tokens a float32 sum takes, and a split that is added to H directly or made of
  // halves keeps that number: weighed at their own, lower cost (a direct split as + 400) fewer and longer splits win, up
  // to five times the tokens in one float32 sum, for less time but a larger distance from the float64 Gram matrix
  // (n = 4096, 16384 tokens: 312 and 250 us, 8.7e-8 and 7.1e-7; n = 9472, 40000: 2881 and 2820 us, 1.8e-7 and 1.2e-6;
  // n = 2048, 2048: 40.7 and 32.2 us, 3.0e-8 and 5.3e-8).
  p.halves = big && ceil_div((int64_t)p.ntb * p.ntb * p.splits_total, 256) * kHalfCost <
                        ceil_div((int64_t)p.ntiles * p.splits_total, 256) * 100;
  p.tile_bytes = (size_t)p.tile * p.tile * ((dt == PTQ_BF16) ? sizeof(float) : sizeof(double));
  int64_t sl = big ? (int64_t)(kMaxPartialBytes / (p.tile_bytes * p.ntiles)) : ceil_div(2048, p.ntiles);
  if (sl > p.splits_total) sl = p.splits_total;
  if (sl < 1) sl = 1;
  p.splits_launch = (int)sl;
  return p;
}

}  // namespace

size_t hessian_workspace_bytes(int64_t n, int64_t t) {
  // sized for either input type and either bf16 kernel
  size_t need = 0;
  for (int v = 0; v < 3; ++v) {
    const Plan p = make_plan(n, t, v == 2 ? PTQ_F32 : PTQ_BF16, v == 0);
    const size_t b = p.tile_bytes * p.ntiles * p.splits_launch;
    if (b > need) need = b;
  }
  return align_up(need, 256);
}

ptq_status hessian_launch(double* H, int64_t ldh, const void* X, ptq_dtype xdt, int64_t t, int64_t n,
                          int64_t ldx, void* ws, size_t ws_bytes, hipStream_t st) {
  if (t == 0 || n == 0) return PTQ_OK;
  const Plan p = make_plan(n, t, xdt, big_kernel_fits(ldx));
  if (ws_bytes < p.tile_bytes * p.ntiles * p.splits_launch) return PTQ_ERR_WORKSPACE;
  for (int s0 = 0; s0 < p.splits_total; s0 += p.splits_launch) {
    const int ns = (p.splits_total - s0 < p.splits_launch) ? p.splits_total - s0 : p.splits_launch;
    const int64_t tok0 = (int64_t)s0 * p.chunk;
    dim3 g((unsigned)p.ntiles, (unsigned)ns);
    dim3 gr((unsigned)p.ntiles, (unsigned)(p.tile * p.tile / 1024));
    if (xdt == PTQ_BF16 && p.tile == kBT) {
      const bool direct = p.splits_total == 1;
      auto launch = [&](auto halves, auto shared, auto direct_) {
        constexpr bool HALVES = decltype(halves)::value, SHARED = decltype(shared)::value, DIRECT = decltype(direct_)::value;
        if (!lds_opt_in<hessian_bf16_big_kernel<HALVES, SHARED, DIRECT>>((int)kBigLdsBytes)) return false;
        const int64_t items = HALVES ? (int64_t)p.ntb * p.ntb : p.ntiles;
        hessian_bf16_big_kernel<HALVES, SHARED, DIRECT><<<256u * (unsigned)ceil_div(items * ns, 256), 256, kBigLdsBytes, st>>>(
            static_cast<const uint16_t*>(X), ldx, t, (int)n, tok0, p.chunk, p.ntb, p.ntiles, ns, static_cast<float*>(ws), H, ldh);
        return true;
      };
      const std::true_type yes;
      const std::false_type no;
      const bool ok = p.halves ? (direct ? launch(yes, yes, yes) : launch(yes, yes, no))
                    : !direct  ? launch(no, no, no)
                    : p.chunk <= kSharedTokens ? launch(no, yes, yes) : launch(no, no, yes);
      if (!ok) return PTQ_ERR_HIP;
      if (!direct)
        hessian_reduce_kernel<float, kBT><<<gr, 256, 0, st>>>(static_cast<const float*>(ws), ns, p.ntiles,
                                                              p.ntb, (int)n, H, ldh);
    } else if (xdt == PTQ_BF16) {
      hessian_bf16_kernel<<<g, 256, 0, st>>>(static_cast<const uint16_t*>(X), ldx, t, (int)n, tok0, p.chunk,
                                             p.ntb, static_cast<float*>(ws));
      hessian_reduce_kernel<float, kTile><<<gr, 256, 0, st>>>(static_cast<const float*>(ws), ns, p.ntiles,
                                                              p.ntb, (int)n, H, ldh);
    } else {
      if (!hessian_f32_partials_launch(static_cast<const float*>(X), ldx, t, (int)n, tok0, p.chunk, p.ntb, p.tile, g,
                                       static_cast<double*>(ws), st))
        return PTQ_ERR_HIP;
      if (p.tile == kTile32Wide)
        hessian_reduce_kernel<double, kTile32Wide><<<gr, 256, 0, st>>>(static_cast<const double*>(ws), ns,
                                                                       p.ntiles, p.ntb, (int)n, H, ldh);
      else
        hessian_reduce_kernel<double, kTile32><<<gr, 256, 0, st>>>(static_cast<const double*>(ws), ns,
                                                                   p.ntiles, p.ntb, (int)n, H, ldh);
    }
  }
  PTQ_HIP_CHECK_LAUNCH();
  return PTQ_OK;
}

}  // namespace ptq
