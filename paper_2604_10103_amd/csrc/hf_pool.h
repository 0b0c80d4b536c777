// Pooled means of a block's rows (Eq. 4), shared by the kernels that form them (internal).
#pragma once

#include "hf_common.h"

namespace hf {

// Mean of the rows [r0, r1) of X (rows of D elements from base, which points at the lane's columns), by one wavefront: what the
// lanes with sub = 0 return are the E columns of theirs.
template <typename T, int D>
struct Pool {
  static constexpr int E = Elem<T>::kPer16B;  // elements per 16-byte load
  static constexpr int LPR = D / E;           // lanes covering one row
  static constexpr int RPP = kWave / LPR;     // rows per pass of the wavefront
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
#pragma unroll
    for (int o = LPR; o < kWave; o <<= 1)
#pragma unroll
      for (int e = 0; e < E; ++e) acc[e] += __shfl_xor(acc[e], o, kWave);
    const float inv = 1.0f / (float)(r1 - r0);
#pragma unroll
    for (int e = 0; e < E; ++e) acc[e] *= inv;
  }
};

}  // namespace hf
