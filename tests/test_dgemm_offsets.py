"""The float64 tile GEMM's loads where rows are so long that an offset inside a tile, or down the columns of k, passes 31 bits:
the loop itself, compiled for the host with stand-ins for what it takes from the GPU, reads a sparse mapping with a mark at every
element and nothing anywhere else."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"

_HIP = r"""
#pragma once
#include <math.h>
#include <stddef.h>
#include <stdint.h>
#include <string.h>
#define __device__
#define __host__
#define __global__
#define __forceinline__ inline
struct { int x, y, z; } threadIdx;
inline void __syncthreads() {}
inline float __uint_as_float(uint32_t u) { float f; memcpy(&f, &u, 4); return f; }
inline long long __double_as_longlong(double d) { long long v; memcpy(&v, &d, 8); return v; }
inline double __longlong_as_double(long long v) { double d; memcpy(&d, &v, 8); return d; }
struct __amdgpu_buffer_rsrc_t {};
#define __builtin_amdgcn_make_buffer_rsrc(...) __amdgpu_buffer_rsrc_t{}
#define __builtin_amdgcn_raw_buffer_load_b64(...) 0.0
#define __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, ...) (c)
#define __builtin_amdgcn_sched_group_barrier(...) (void)0
#define __builtin_amdgcn_update_dpp(old, v, ...) (v)
enum { hipSuccess, hipFuncAttributeMaxDynamicSharedMemorySize };
inline int hipGetDevice(int* d) { *d = 0; return 0; }
inline int hipFuncSetAttribute(const void*, int, int) { return 0; }
typedef void* hipStream_t;
struct dim3 {};
inline int hipGetLastError() { return 0; }
"""

_MAIN = r"""
#include "dgemm.h"
#include <stdio.h>
#include <stdlib.h>
#include <sys/mman.h>
using namespace ptq;
static int64_t seen = 0;
static double mark(int o, int k) { return 1.0 + 4096.0 * o + k; }
struct Check {
  int count, kend;
  bool rows_first;
  double operator()(double v, int x, int y) const {
    const int o = rows_first ? x : y, k = rows_first ? y : x;
    if (o < count && k < kend) {
      ++seen;
      if (v != mark(o, k)) { printf("element %d, %d reads %f\n", o, k, v); exit(1); }
    }
    return v;
  }
};
// one operand with the given strides (negative ones run down from the end of the mapping), the other a small dense one
template <int TM, int TN, bool KF, bool SIDE_A>
void run(int64_t so, int64_t sk, int count, int kbeg, int kend) {
  const int64_t span = (count - 1) * llabs(so) + (kend - 1) * llabs(sk) + 1;
  double* m = (double*)mmap(0, span * 8, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (m == MAP_FAILED) { printf("no mapping\n"); exit(2); }
  double* first = m + (so < 0 ? -so * (count - 1) : 0) + (sk < 0 ? -sk * (kend - 1) : 0);
  for (int o = 0; o < count; ++o)
    for (int k = kbeg; k < kend; ++k) first[o * so + k * sk] = mark(o, k);
  static double dense[512 * 128], smem[DgemmTile<TM, TN>::kSmemDoubles];
  using Stride = decltype(DView::so);
  const DView view{first, (Stride)so, (Stride)sk}, other{dense, 1, 128};
  for (int t = 0; t < 256; ++t) {
    threadIdx.x = t;
    f64x4 acc[TM][TN] = {};
    if constexpr (SIDE_A)
      dgemm_mainloop<TM, TN, KF, false>(acc, view, Check{count, kend, true}, other, DgemmIdentity{}, count, 32 * TN, kbeg, kend, smem);
    else
      dgemm_mainloop<TM, TN, false, KF>(acc, other, DgemmIdentity{}, view, Check{count, kend, false}, 32 * TM, count, kbeg, kend, smem);
  }
  munmap(m, span * 8);
}
template <int TM, int TN, bool SIDE_A>
void shapes() {
  constexpr int edge = 32 * (SIDE_A ? TM : TN);
  const int counts[] = {edge, edge - 1, edge - 16, 17, 16, 1}, ranges[][2] = {{0, 256}, {208, 288}, {208, 293}, {240, 257}, {0, 5}};
  for (int c : counts) {
    for (const auto& k : ranges) {
      run<TM, TN, false, SIDE_A>(1, (1 << 23) + 3, c, k[0], k[1]);      // columns of k down long rows
      run<TM, TN, false, SIDE_A>(-1, -(1 << 23) - 3, c, k[0], k[1]);
      run<TM, TN, true, SIDE_A>((1 << 25) + 5, 1, c, k[0], k[1]);       // long rows themselves
      run<TM, TN, true, SIDE_A>(-(1 << 25) - 5, -1, c, k[0], k[1]);
    }
    run<TM, TN, true, SIDE_A>((int64_t{3} << 30) + 1, 1, c < 5 ? c : 5, 0, 20);   // a stride past 31 bits itself
  }
}
int main() {
  shapes<1, 1, true>(); shapes<1, 1, false>(); shapes<2, 2, true>(); shapes<2, 2, false>();
  shapes<2, 4, true>(); shapes<2, 4, false>(); shapes<4, 4, true>(); shapes<4, 4, false>();
  printf("%lld\n", (long long)seen);
}
"""


@pytest.mark.skipif(not os.path.exists(CLANG), reason="needs the host side of the ROCm compiler")
def test_offsets_past_31_bits(tmp_path):
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(_HIP)
    (tmp_path / "main.cpp").write_text(_MAIN)
    exe = str(tmp_path / "check")
    subprocess.run([CLANG, "-x", "c++", "-std=c++17", "-O1", "-w", "-I", str(tmp_path), "-I",
                    os.path.join(ROOT, "paper_2601_19675_amd", "csrc"), str(tmp_path / "main.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.returncode, r.stdout[-300:])
    assert int(r.stdout.split()[-1]) > 100000
