// Linear state of the history branch: zero fill and absorption of evicted tokens (Eq. 2).
//
//   L[i][j] += sum_t R_t(phi(k_t))[i] * v_t[j]        z[i] += sum_t phi(k_t)[i]
//
// This file: the fill kernel and the fp32-arithmetic absorb kernel (fp32 inputs, or head_dim 64).
// bf16 inputs with head_dim 128 take the MFMA kernel of hf_state_mfma.hip.
#include <type_traits>

#include "hf_absorb_wide.h"

namespace hf {

__global__ void fill_zero_kernel(float* __restrict__ p, size_t n) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = 0.0f;
}

int launch_fill_zero(float* p, size_t n, hipStream_t s) {
  const int threads = 256;
  size_t blocks = (n + threads - 1) / threads;
  if (blocks > 2048) blocks = 2048;
  hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)blocks), dim3(threads), 0, s, p, n);
  return check_launch("hf_state_init");
}

// ---------------------------------------------------------------------------------------------
// Linear map of Eq. 3 folded into the state: L'[bh] = L[bh] W[h], z' = z.  Runs once per chunk on
// 0.8 MB, fp32 FMA: one workgroup per 16 rows of one head's L; thread (row, column group) forms 8
// (or 4) output columns; the 16 rows of L sit in LDS (broadcast reads), W streams from L2 with
// the 16 column groups of a row reading 512 (256) contiguous bytes.
template <int D>
__global__ __launch_bounds__(256) void fold_linear_kernel(const float* __restrict__ state_in,
                                                          const float* __restrict__ W,
                                                          float* __restrict__ state_out, int H, int BH) {
  constexpr int C = D / 16;  // output columns per thread
  __shared__ float sL[16][D];
  const int tid = threadIdx.x, row = tid >> 4, cg = tid & 15;
  const int bh = blockIdx.y, h = bh % H, i0 = blockIdx.x * 16;
  const float* Lin = state_in + (size_t)bh * D * D + (size_t)i0 * D;
  for (int e = tid; e < 16 * D; e += 256) sL[e / D][e % D] = Lin[e];
  if (blockIdx.x == 0 && tid < D)  // the normaliser is copied unchanged
    state_out[(size_t)BH * D * D + (size_t)bh * D + tid] = state_in[(size_t)BH * D * D + (size_t)bh * D + tid];
  __syncthreads();
  const float* Wh = W + (size_t)h * D * D + cg * C;
  float acc[C];
#pragma unroll
  for (int c = 0; c < C; ++c) acc[c] = 0.0f;
#pragma unroll 4
  for (int j = 0; j < D; ++j) {
    const float l = sL[row][j];
    float w[C];
#pragma unroll
    for (int c = 0; c < C; c += 4) {
      const float4 v = *reinterpret_cast<const float4*>(Wh + (size_t)j * D + c);
      w[c] = v.x; w[c + 1] = v.y; w[c + 2] = v.z; w[c + 3] = v.w;
    }
#pragma unroll
    for (int c = 0; c < C; ++c) acc[c] = fmaf(l, w[c], acc[c]);
  }
  float* out = state_out + (size_t)bh * D * D + (size_t)(i0 + row) * D + cg * C;
#pragma unroll
  for (int c = 0; c < C; c += 4) *reinterpret_cast<float4*>(out + c) = make_float4(acc[c], acc[c + 1], acc[c + 2], acc[c + 3]);
}

int launch_fold_linear(const hf_config& c, const float* state_in, const float* W, float* state_out, hipStream_t s) {
  const int BH = c.batch * c.heads;
  const dim3 grid(c.head_dim / 16, BH), block(256);
  if (c.head_dim == 128)
    hipLaunchKernelGGL((fold_linear_kernel<128>), grid, block, 0, s, state_in, W, state_out, c.heads, BH);
  else
    hipLaunchKernelGGL((fold_linear_kernel<64>), grid, block, 0, s, state_in, W, state_out, c.heads, BH);
  return check_launch("hf_state_fold_linear");
}

// ---------------------------------------------------------------------------------------------
// fp32 arithmetic (fp32 inputs, or head_dim 64), a launch of its own: see absorb_tile
template <typename T, int D>
__global__ __launch_bounds__(64 * kAbsorbWaves) void absorb_wide_kernel(const float* state_in, float* state_out,
                                                                        const T* __restrict__ K, const T* __restrict__ V,
                                                                        int n, int head_stride, int per,
                                                                        const float* __restrict__ cosv,
                                                                        const float* __restrict__ sinv, int phi_kind, int BH,
                                                                        int one_slice) {
  constexpr int TILES = (D / 32) * (D / 32);
  __shared__ float smem[kAbsorbLds / sizeof(float)];
  absorb_tile<T, D>(smem, blockIdx.x % TILES, blockIdx.x / TILES, blockIdx.y, state_in, state_out, K, V, n, head_stride, per, cosv,
                    sinv, phi_kind, BH, one_slice);
}

// state_in NULL: an empty state.  More than one slice needs state_in == state_out.
template <typename T, int D>
static int launch_absorb_wide(const hf_config& c, const float* state_in, float* state_out, const void* K, const void* V, int n,
                              int head_stride, const float* cosv, const float* sinv, hipStream_t s) {
  constexpr int TILES = (D / 32) * (D / 32);
  const int BH = c.batch * c.heads;
  // one slice for a chunk of a small stream; else four workgroups per compute unit, 256 tokens per slice or more
  int slices = 1;
  if (n > kAbsorbOneSlice) {
    slices = (1024 + TILES * BH - 1) / (TILES * BH);
    if (slices > (n + 255) / 256) slices = (n + 255) / 256;
  }
  const int per = ((n + slices - 1) / slices + kAbsorbRun - 1) / kAbsorbRun * kAbsorbRun;
  slices = (n + per - 1) / per;
  hipLaunchKernelGGL((absorb_wide_kernel<T, D>), dim3(slices * TILES, BH), dim3(64 * kAbsorbWaves), 0, s, state_in, state_out,
                     static_cast<const T*>(K), static_cast<const T*>(V), n, head_stride, per, cosv, sinv, c.phi, BH, slices == 1);
  return check_launch("hf_absorb_evicted");
}

static int launch_absorb_fp32(const hf_config& c, const float* state_in, float* state_out, const void* K, const void* V, int n,
                              int head_stride, const float* cosv, const float* sinv, hipStream_t s) {
  if (c.dtype == HF_F32)
    return c.head_dim == 128 ? launch_absorb_wide<float, 128>(c, state_in, state_out, K, V, n, head_stride, cosv, sinv, s)
                             : launch_absorb_wide<float, 64>(c, state_in, state_out, K, V, n, head_stride, cosv, sinv, s);
  return launch_absorb_wide<bf16_t, 64>(c, state_in, state_out, K, V, n, head_stride, cosv, sinv, s);
}

int launch_absorb_mfma(const hf_config& c, float* state, const void* K, const void* V, int n, int head_stride,
                       const float* cosv, const float* sinv, void* workspace, size_t workspace_bytes,
                       hipStream_t s, void* planes_out);  // hf_state_mfma.hip
size_t absorb_mfma_workspace_bytes(const hf_config& c, int n);

static bool absorb_uses_mfma(const hf_config& c) { return c.dtype == HF_BF16 && c.head_dim == 128; }

size_t absorb_workspace_bytes(const hf_config& c, int n) {
  return absorb_uses_mfma(c) ? absorb_mfma_workspace_bytes(c, n) : 0;
}

// planes_out != NULL (bf16, head_dim 128 only; the caller checks): the bf16 planes of the updated state as well
int launch_absorb(const hf_config& c, float* state, const void* K, const void* V, int n, int head_stride,
                  const float* cosv, const float* sinv, void* workspace, size_t workspace_bytes,
                  hipStream_t s, void* planes_out) {
  if (absorb_uses_mfma(c))
    return launch_absorb_mfma(c, state, K, V, n, head_stride, cosv, sinv, workspace, workspace_bytes, s, planes_out);
  return launch_absorb_fp32(c, state, state, K, V, n, head_stride, cosv, sinv, s);
}

// state_out = state_in (NULL: an empty state) + the tokens' contribution; the buffers do not overlap
int launch_absorb_into(const hf_config& c, const float* state_in, float* state_out, const void* K, const void* V, int n,
                       int head_stride, const float* cosv, const float* sinv, void* workspace, size_t workspace_bytes,
                       hipStream_t s) {
  if (!absorb_uses_mfma(c) && n <= kAbsorbOneSlice)
    return launch_absorb_fp32(c, state_in, state_out, K, V, n, head_stride, cosv, sinv, s);
  const size_t count = (size_t)c.batch * c.heads * c.head_dim * (c.head_dim + 1);
  if (state_in) {
    if (hipMemcpyAsync(state_out, state_in, count * sizeof(float), hipMemcpyDeviceToDevice, s) != hipSuccess) {
      set_error("copy of the state: %s", hipGetErrorString(hipGetLastError()));
      return HF_ERR_HIP;
    }
  } else {
    const int rc = launch_fill_zero(state_out, count, s);
    if (rc != HF_OK) return rc;
  }
  return launch_absorb(c, state_out, K, V, n, head_stride, cosv, sinv, workspace, workspace_bytes, s);
}

// ---------------------------------------------------------------------------------------------
// Window compaction after an eviction: tokens [src, src + len) of every head move to [dst, dst + len)
// in K_win and V_win (16-byte pieces; blockIdx.z picks K or V).  The caller issues non-overlapping
// pieces in ascending order, so a launch never reads what it writes.
__global__ __launch_bounds__(256) void window_shift_kernel(uint4* __restrict__ K, uint4* __restrict__ V,
                                                           size_t head_stride16, size_t src16, size_t dst16,
                                                           size_t len16) {
  uint4* X = (blockIdx.z ? V : K) + (size_t)blockIdx.y * head_stride16;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < len16; i += (size_t)gridDim.x * 256)
    X[dst16 + i] = X[src16 + i];
}

int launch_window_shift(const hf_config& c, void* K, void* V, int n_kv, int first, int n_evict, hipStream_t s) {
  const int BH = c.batch * c.heads;
  const size_t row16 = (size_t)c.head_dim * (c.dtype == HF_BF16 ? 2 : 4) / 16;  // 16-byte pieces per token
  const int keep = n_kv - first - n_evict;  // tokens behind the evicted run move down to `first`
  // pieces of at most n_evict tokens: source [t + n_evict, ...) and destination [t, ...) never overlap
  for (int t = 0; t < keep; t += n_evict) {
    const int len = min(n_evict, keep - t);
    const size_t len16 = (size_t)len * row16;
    unsigned blocks = (unsigned)((len16 + 255) / 256);
    if (blocks > 1024) blocks = 1024;
    hipLaunchKernelGGL(window_shift_kernel, dim3(blocks, BH, 2), dim3(256), 0, s, static_cast<uint4*>(K),
                       static_cast<uint4*>(V), (size_t)kv_stride_of(c, n_kv) * row16,
                       (size_t)(first + t + n_evict) * row16, (size_t)(first + t) * row16, len16);
    const int rc = check_launch("hf_window_advance(shift)");
    if (rc != HF_OK) return rc;
  }
  return HF_OK;
}

}  // namespace hf
