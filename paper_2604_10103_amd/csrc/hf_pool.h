// Pooled means of a block's rows (Eq. 4), shared by the kernels that form them, and what selecting kernels begin with (internal).
#pragma once

#include "hf_common.h"

namespace hf {

// A kernel's arguments of at least 64 (kLines - 1) + 4 bytes (hidden ones not counted) span kLines lines of the scalar cache.  The compiler loads each where it is
// used, so a workgroup's chain stood still at every line it met for the first time; here all of them are fetched together, with the
// first (3 heads x 400 queries over four steps 61.8 -> 60.3 us).  A dense window's launch has nothing to win by it (40 heads x 576:
// 29.0 -> 29.5).
template <int kLines>
__device__ __forceinline__ void warm_arguments() {
  static_assert(kLines == 4 || kLines == 5, "four or five lines");
  const void* const args = (const void*)__builtin_amdgcn_kernarg_segment_ptr();
  int t0, t1, t2, t3, t4;
  if constexpr (kLines == 5)
    asm volatile("s_load_dword %0, %5, 0x0\n\ts_load_dword %1, %5, 0x40\n\ts_load_dword %2, %5, 0x80\n\ts_load_dword %3, %5, 0xc0\n\t"
                 "s_load_dword %4, %5, 0x100\n\ts_waitcnt lgkmcnt(0)"
                 : "=&s"(t0), "=&s"(t1), "=&s"(t2), "=&s"(t3), "=&s"(t4) : "s"(args));
  else
    asm volatile("s_load_dword %0, %4, 0x0\n\ts_load_dword %1, %4, 0x40\n\ts_load_dword %2, %4, 0x80\n\ts_load_dword %3, %4, 0xc0\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&s"(t0), "=&s"(t1), "=&s"(t2), "=&s"(t3) : "s"(args));
  // (awaited in their block; read as well, as an output that nobody reads counts as free)
  asm volatile("" :: "s"(t0), "s"(t1), "s"(t2), "s"(t3));
  if constexpr (kLines == 5) asm volatile("" :: "s"(t4));
}

// Mean of the rows [r0, r1) of X (rows of D elements from base, which points at the lane's columns), by one wavefront: what the
// lanes with sub = 0 return are the E columns of theirs.
template <typename T, int D>
struct Pool {
  static constexpr int E = Elem<T>::kPer16B;  // elements per 16-byte load
  static constexpr int LPR = D / E;           // lanes covering one row
  static constexpr int RPP = kWave / LPR;     // rows per pass of the wavefront
  // kVector: how the lanes' sums meet, see finish
  template <bool kVector>
  static __device__ __forceinline__ void mean(const T* __restrict__ base, int r0, int r1, int sub, float (&acc)[E]) {
#pragma unroll
    for (int e = 0; e < E; ++e) acc[e] = 0.0f;
    int r = r0 + sub;
    // sixteen, then eight independent 16-byte loads in flight per lane
    for (; r + 15 * RPP < r1; r += 16 * RPP) {
      float v[16][E];
#pragma unroll
      for (int u = 0; u < 16; ++u) load16B<T>(base + (size_t)(r + u * RPP) * D, v[u]);
#pragma unroll
      for (int u = 0; u < 16; ++u)
#pragma unroll
        for (int e = 0; e < E; ++e) acc[e] += v[u][e];
    }
    for (; r + 7 * RPP < r1; r += 8 * RPP) {
      float v[8][E];
#pragma unroll
      for (int u = 0; u < 8; ++u) load16B<T>(base + (size_t)(r + u * RPP) * D, v[u]);
#pragma unroll
      for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int e = 0; e < E; ++e) acc[e] += v[u][e];
    }
    if (r < r1) {   // fewer than eight rows left: requested together all the same (clamped rows are dropped)
      float v[8][E];
#pragma unroll
      for (int u = 0; u < 8; ++u) load16B<T>(base + (size_t)min(r + u * RPP, r1 - 1) * D, v[u]);
#pragma unroll
      for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int e = 0; e < E; ++e) acc[e] += r + u * RPP < r1 ? v[u][e] : 0.0f;
    }
    finish<kVector>(r1 - r0, acc);
  }
  // The same mean of at most kFew rows in two halves, so that the rows of several blocks can be requested before the first is summed.
  static constexpr int kFew = 8 * RPP;
  static __device__ __forceinline__ void request(const T* __restrict__ base, int r0, int r1, int sub, float (&v)[8][E]) {
#pragma unroll
    for (int u = 0; u < 8; ++u) load16B<T>(base + (size_t)min(r0 + sub + u * RPP, r1 - 1) * D, v[u]);
  }
  static __device__ __forceinline__ void mean_of(const float (&v)[8][E], int r0, int r1, int sub, float (&acc)[E]) {
#pragma unroll
    for (int e = 0; e < E; ++e) acc[e] = 0.0f;
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int e = 0; e < E; ++e) acc[e] += r0 + sub + u * RPP < r1 ? v[u][e] : 0.0f;
    finish<true>(r1 - r0, acc);
  }

 private:
  // Rows of sixteen and halves of the wavefront by the vector unit where a chain of steps waits for the sum (through the LDS each of
  // them is a round trip); launches that do nothing but pool have other wavefronts to run meanwhile and the vector unit busy with
  // sums: there through the LDS (fp32, 3 heads of 128, 922 x 2766: selection 7.35 us by the vector unit, 7.23 so).
  template <bool kVector>
  static __device__ __forceinline__ void finish(int rows, float (&acc)[E]) {
#pragma unroll
    for (int o = LPR; o < kWave; o <<= 1)
#pragma unroll
      for (int e = 0; e < E; ++e) {
        if (!kVector || o < 16) {
          acc[e] += __shfl_xor(acc[e], o, kWave);
        } else {
          const uint32_t a = __float_as_uint(acc[e]);
          const auto sw = o == 16 ? __builtin_amdgcn_permlane16_swap(a, a, false, false) : __builtin_amdgcn_permlane32_swap(a, a, false, false);
          acc[e] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
        }
      }
    const float inv = 1.0f / (float)rows;
#pragma unroll
    for (int e = 0; e < E; ++e) acc[e] *= inv;
  }
};

}  // namespace hf
