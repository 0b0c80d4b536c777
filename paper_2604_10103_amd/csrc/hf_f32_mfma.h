// Building blocks of the fp32-arithmetic kernels on the fp32 matrix instruction v_mfma_f32_16x16x4_f32 (internal).
//
// The instruction multiplies A (16 x 4) by B (4 x 16): lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16] and holds
// C[4 (l / 16) + r][l % 16], r = 0..3.  The four k indices of one instruction may be any four as long as A and B agree,
// so both operands come as 16-byte pieces of row-major memory, and one piece feeds four instructions:
//
//   row form     lane l holds X[row l % 16][16 c + 4 (l / 16) .. + 4): the piece's elements are k = 4 (l / 16) + e of the
//                four instructions e = 0..3: products over FEATURES (A and B alike)
//   column form  lane l holds X[token 4 (l / 16) + r][64 f + 4 (l % 16) .. + 4): instruction r has k = token 4 (l / 16) + r,
//                and the piece's elements are four different 16-row operands (features 64 f + 4 i + e): products over
//                TOKENS, whose B operand is exactly the C layout of a row-form product (token 4 (l / 16) + r of column l % 16)
//
// An accumulator of a column-form product (f, e) holds features 64 f + 16 (l / 16) + 4 r + e of column l % 16: for fixed r
// the four e are consecutive.  Nothing passes through LDS: a wavefront reads its operands straight from memory (L1, L2)
// one tile ahead, and 32 cycles of matrix work per kilobyte requested leave the caches half idle.
//
// The 32 x 32 x 2 instruction works the same way with 32 rows and columns and two k indices: lane l supplies
// A[l % 32][l / 32], a row-form piece is X[row l % 32][8 c + 4 (l / 32) .. + 4), C's register r is row
// 8 (r / 4) + 4 (l / 32) + r % 4, and a column-form piece of a token covers 4 x 32 (or 2 x 32) features.
// Vector instructions between fp32 matrix instructions are not hidden by them on this chip (probe, two wavefronts per SIMD,
// TFLOP/s of the chip): 16x16x4 alone 144, with one v_fma behind each 125, with four 106; 32x32x2 alone 154, with one for
// each 2048 flops 132.  So the wide tile is taken where the blocks allow it: half the vector work per product, and twice
// the products per kilobyte requested.
#pragma once

#include "hf_common.h"

namespace hf {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// what the attention kernels that add the history term from the fp32 state take for it
struct WideHist {            // history term, or statistics for the backward pass
  const float* L;            // [BH][D][D], NULL: none
  const float* z;            // [BH][D]
  const float* cosq;         // [n_q][D/2] rotation of phi(q) in the numerator, or NULL
  const float* sinq;
  const void* q_hist;        // [BH][n_q][D] queries of the history branch
  float eps, z_scale;
  int phi_kind;
  float* lse2;               // [BH][n_q], given: row statistics instead of an output
  const void* d_out;         // [BH][n_q][D]
  float* dvec;               // [BH][n_q] d_out . O_local
};

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ f32x16 mfma_f32_wide(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// four consecutive elements as fp32
template <typename T> __device__ __forceinline__ f32x4 load4(const T* p);
template <> __device__ __forceinline__ f32x4 load4<float>(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
template <> __device__ __forceinline__ f32x4 load4<bf16_t>(const bf16_t* p) {
  const uint2 w = *reinterpret_cast<const uint2*>(p);
  return f32x4{__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u), __uint_as_float(w.y << 16),
               __uint_as_float(w.y & 0xffff0000u)};
}
template <typename T> __device__ __forceinline__ void store4(T* p, f32x4 v);
template <> __device__ __forceinline__ void store4<float>(float* p, f32x4 v) { *reinterpret_cast<f32x4*>(p) = v; }
template <> __device__ __forceinline__ void store4<bf16_t>(bf16_t* p, f32x4 v) {
  uint2 w;
  w.x = pack_bf16(v[0], v[1]);
  w.y = pack_bf16(v[2], v[3]);
  *reinterpret_cast<uint2*>(p) = w;
}

// tokens first .. first + cnt - 1 of a head (whole wavefronts agree on them) as a buffer: rows behind them read as zeros.  A
// real row in their place would pass a NaN or an infinity on to rows that have nothing to do with it, also with weight zero.
template <typename T, int D>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rows(const T* head, int first, int cnt) {
  const T* p = head + (size_t)__builtin_amdgcn_readfirstlane(first) * D;
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(p), 0, __builtin_amdgcn_readfirstlane(cnt) * D * (int)sizeof(T), 0x00020000);
}

// what a lane keeps of the memory it asked for (four elements, at a byte offset): the storage type's own
// words, widened when they are used, so that a tile on its way takes no more registers than it has bytes
template <typename T> struct Piece;
template <> struct Piece<float> {
  f32x4 v;
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rows, int at) {
    v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rows, at, 0, 0));
  }
  __device__ __forceinline__ f32x4 get() const { return v; }
};
template <> struct Piece<bf16_t> {
  uint2 w;
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rows, int at) {
    w = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(rows, at, 0, 0));
  }
  __device__ __forceinline__ f32x4 get() const {
    return f32x4{__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u), __uint_as_float(w.y << 16),
                 __uint_as_float(w.y & 0xffff0000u)};
  }
};

// sum / maximum over the four lanes l % 16, + 16, + 32, + 48 that share a column: two register swaps between rows of
// lanes (vector instructions; a lane exchange through LDS would be a round trip of a hundred cycles)
__device__ __forceinline__ float column_sum(float v) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}
__device__ __forceinline__ float column_max(float v) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// adjacent feature pairs of four consecutive features turned by two angles
__device__ __forceinline__ f32x4 rotate4(f32x4 x, float c0, float s0, float c1, float s1) {
  return f32x4{x[0] * c0 - x[1] * s0, x[0] * s0 + x[1] * c0, x[2] * c1 - x[3] * s1, x[2] * s1 + x[3] * c1};
}

// workgroups of `rows` rows of a query block that have a row: what the launch rules count.  (A block longer than
// n_q, or the end of the last one, has workgroups without any; they return at once.)
inline long long row_groups(const hf_config& c, int n_q, int rows) {
  return (long long)c.batch * c.heads * ((long long)(n_q / c.block_q) * ((c.block_q + rows - 1) / rows) + (n_q % c.block_q + rows - 1) / rows);
}

}  // namespace hf
