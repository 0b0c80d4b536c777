// Eq. 2 in fp32 arithmetic by one workgroup: a tile of the state over a slice of the tokens (internal).
#pragma once

#include <type_traits>

#include "hf_f32_mfma.h"

namespace hf {

// fp32 arithmetic (fp32 inputs, or head_dim 64): the contraction over tokens on the fp32 matrix instruction.
// v_mfma_f32_32x32x2 multiplies 32 features of phi(k) by 32 features of v over two tokens, and lane l supplies feature
// l % 32 of token l / 32 of both: operands come straight from memory, 128 contiguous bytes per token.  A workgroup owns one
// 32 x 32 tile of L and a slice of the tokens; its eight wavefronts take every eighth run of 16 tokens, the loads of the next
// run in flight under the products of the current one, and meet in LDS.
// Eight wavefronts on one compute unit are bound by their issue, so a round has no branch, mask or address per token (1000
// tokens of one head of 64, plain / rotated: 9.6 / 12.2 us; 14.7 / 16.9 with them, more than the 12.7 / 13.2 before).
// A chunk of a small stream is one slice: the tile is then written as state_in + sum by plain stores, into another buffer
// if the caller wants, where more slices add to the state with float atomics (state_in == state_out).
// Latency-bound at the sizes of fp32 streams.  256 threads per (head, 64 tokens or more) with FMA arithmetic, tokens staged
// through LDS and atomics took 12.2 us for 2 heads of 64 with 64 tokens, behind a copy of the state of 1.5 us; this kernel
// 3.9 us, without a copy (ring of 2 heads of 64, window of 256: 37 -> 27 us a chunk).
constexpr int kAbsorbWaves = 8;
constexpr int kAbsorbRun = 16 * kAbsorbWaves;   // tokens per round of the workgroup
constexpr int kAbsorbOneSlice = 1024;           // up to eight rounds (one head of 64: 9.6 us; slices and atomics took 12.7 with FMA)

constexpr int kAbsorbLds = kAbsorbWaves * (32 * 32 + 32) * (int)sizeof(float);   // bytes

// smem: kAbsorbLds bytes; 64 kAbsorbWaves threads
template <typename T, int D>
__device__ __forceinline__ void absorb_tile(float* smem, int tile, int slice, int bh, const float* state_in, float* state_out,
                                            const T* __restrict__ K, const T* __restrict__ V, int n, int head_stride, int per,
                                            const float* __restrict__ cosv, const float* __restrict__ sinv, int phi_kind, int BH,
                                            int one_slice) {
  constexpr int TS = D / 32;                    // tiles per side of L
  auto part = reinterpret_cast<float(*)[32][32]>(smem);
  auto zpart = reinterpret_cast<float(*)[32]>(smem + kAbsorbWaves * 32 * 32);
  const int it = tile / TS, jt = tile % TS;
  const int t0 = slice * per, t1 = min(n, t0 + per);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, h = lane >> 5;
  const int fi = 32 * it + l32, fj = 32 * jt + l32;
  const T* Kh = K + (size_t)bh * head_stride * D + fi;  // head_stride tokens between heads (= n when packed)
  const T* Vh = V + (size_t)bh * head_stride * D + fj;
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
  float zsum = 0.0f;
  T kr[8], vr[8];
  float cs[8], sn[8];
  // a whole run at offsets from one address, without masks: with them address and mask arithmetic is most of a round
  auto load = [&](int base) {
    if (base + 16 <= t1) {                      // uniform
      const T *kp = Kh + (size_t)(base + h) * D, *vp = Vh + (size_t)(base + h) * D;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        kr[u] = kp[2 * u * D];
        vr[u] = vp[2 * u * D];
      }
      if (cosv) {
        const size_t at = (size_t)(base + h) * (D / 2) + fi / 2;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          cs[u] = cosv[at + u * D];
          sn[u] = sinv[at + u * D];
        }
      }
    } else {
#pragma unroll
      for (int u = 0; u < 8; ++u) {             // tokens past the slice: clamped addresses, zeroed below
        const size_t t = (size_t)min(base + 2 * u + h, t1 - 1);
        kr[u] = Kh[t * D];
        vr[u] = Vh[t * D];
        if (cosv) {
          cs[u] = cosv[t * (D / 2) + fi / 2];
          sn[u] = sinv[t * (D / 2) + fi / 2];
        }
      }
    }
  };
  float a[8], b[8];
  auto operands = [&](int base, auto whole) {   // (each choice once for all eight: a branch per token keeps them apart)
    auto real = [&](int u) { return whole.value || base + 2 * u + h < t1; };
    if (phi_kind == HF_PHI_RELU) {
#pragma unroll
      for (int u = 0; u < 8; ++u) a[u] = phi_apply(Elem<T>::load(&kr[u]), HF_PHI_RELU);
    } else {
#pragma unroll
      for (int u = 0; u < 8; ++u) a[u] = phi_apply(Elem<T>::load(&kr[u]), HF_PHI_ELU1);
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      a[u] = real(u) ? a[u] : 0.0f;
      b[u] = real(u) ? Elem<T>::load(&vr[u]) : 0.0f;
      zsum += a[u];                             // the normaliser takes the un-rotated phi(k)
    }
    if (cosv) {                                 // pairs (2 p, 2 p + 1) are neighbouring lanes
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const float other = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(a[u]), 0xb1, 0xf, 0xf, false));   // lane ^ 1
        const float x = (l32 & 1) ? other * sn[u] + a[u] * cs[u] : a[u] * cs[u] - other * sn[u];
        a[u] = real(u) ? x : 0.0f;
      }
    }
  };
  int base = t0 + 16 * wave;
  if (base < t1) load(base);
  for (; base < t1; base += kAbsorbRun) {
    if (base + 16 <= t1) operands(base, std::true_type{}); else operands(base, std::false_type{});
    if (base + kAbsorbRun < t1) load(base + kAbsorbRun);
#pragma unroll
    for (int u = 0; u < 8; ++u) acc = mfma_f32_wide(a[u], b[u], acc);
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) part[wave][8 * (r >> 2) + 4 * h + (r & 3)][l32] = acc[r];
  zsum += __shfl_xor(zsum, 32, kWave);
  if (h == 0) zpart[wave][l32] = zsum;
  __syncthreads();
  const size_t at = (size_t)bh * D * D + (size_t)(32 * it) * D + 32 * jt;
  for (int e = threadIdx.x; e < 1024; e += 64 * kAbsorbWaves) {
    const int i = e >> 5, j = e & 31;
    float v = 0.0f;
#pragma unroll
    for (int w = 0; w < kAbsorbWaves; ++w) v += part[w][i][j];
    const size_t x = at + (size_t)i * D + j;
    if (one_slice) state_out[x] = (state_in ? state_in[x] : 0.0f) + v;
    else atomicAdd(state_out + x, v);
  }
  if (jt == 0 && threadIdx.x < 32) {
    float v = 0.0f;
#pragma unroll
    for (int w = 0; w < kAbsorbWaves; ++w) v += zpart[w][threadIdx.x];
    const size_t x = (size_t)BH * D * D + (size_t)bh * D + 32 * it + threadIdx.x;
    if (one_slice) state_out[x] = (state_in ? state_in[x] : 0.0f) + v;
    else atomicAdd(state_out + x, v);
  }
}

}  // namespace hf
