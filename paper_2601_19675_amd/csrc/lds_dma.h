// Requests that bring data from memory straight into LDS (buffer_load ... lds), issued by inline assembly and waited for
// by count: for its own the compiler waits for all of them before each LDS read.  Not part of the C ABI.
//
// The compiler does not look into inline assembly for the wait states that an instruction needs after the one that
// wrote its scalar operands, so they stand here: one between a scalar write of m0 and the request that takes its LDS
// address from it, five between a vector instruction that writes a scalar register (readfirstlane) and a request that has it
// in its descriptor or offset.  build.py checks both on the generated assembly.
#pragma once
#include <type_traits>
#include <utility>

#include "common.h"

namespace ptq {

typedef __attribute__((__vector_size__(4 * sizeof(int)))) int i32x4;

// a buffer of `bytes` (below 2^32) at p; p and bytes the same for a wave
__device__ __forceinline__ i32x4 buffer_at(const void* p, int64_t bytes) {
  const uint64_t a = (uint64_t)p;
  i32x4 b{(int)__builtin_amdgcn_readfirstlane((uint32_t)a), (int)__builtin_amdgcn_readfirstlane((uint32_t)(a >> 32)),
          (int)__builtin_amdgcn_readfirstlane((uint32_t)(bytes > 0 ? bytes : 0)), 0x00020000};
  asm volatile("s_nop 4" : "+s"(b));   // behind the readfirstlanes
  return b;
}

// 64 lanes x 16, 4 or 1 bytes from descriptor base + voff + soff to LDS address ldsaddr + 16 or 4 lane; lanes past the
// descriptor's end deliver zeros.  (Nothing else in these kernels uses m0: no indirect register indexing.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int BYTES>
__device__ __forceinline__ void request_to_lds(i32x4 rsrc, uint32_t voff, uint32_t soff, uint32_t ldsaddr) {
  static_assert(BYTES == 16 || BYTES == 4 || BYTES == 1, "");
  if constexpr (BYTES == 16)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(ldsaddr), "v"(voff), "s"(rsrc), "s"(soff)
                 : "memory", "m0");
  else if constexpr (BYTES == 4)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, %3 offen lds" ::"s"(ldsaddr), "v"(voff), "s"(rsrc), "s"(soff)
                 : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_ubyte %1, %2, %3 offen lds" ::"s"(ldsaddr), "v"(voff), "s"(rsrc), "s"(soff)
                 : "memory", "m0");
}

// 16 bytes a lane, no scalar offset
__device__ __forceinline__ void request_to_lds(i32x4 rsrc, uint32_t voff, uint32_t ldsaddr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(ldsaddr), "v"(voff), "s"(rsrc)
               : "memory", "m0");
}

// The same with the LDS address as a scalar base plus a compile-time offset: one scalar instruction per request
// instead of an add into a temporary and a move.
template <uint32_t OFFSET>
__device__ __forceinline__ void request_to_lds_at(i32x4 rsrc, uint32_t voff, uint32_t ldsbase) {
  asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(ldsbase), "v"(voff), "s"(rsrc),
               "n"(OFFSET)
               : "memory", "m0", "scc");
}
#pragma clang diagnostic pop

// until N requests to memory are on their way; the other counters: no wait
template <int N>
__device__ __forceinline__ void wait_requests() {
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0f70);
}

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>)
template <class F, int... Is>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, Is...>) {
  (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

}  // namespace ptq
