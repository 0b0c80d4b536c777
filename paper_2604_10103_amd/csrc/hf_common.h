// Shared host/device helpers of the gfx950 hybrid-attention library (internal).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "hf.h"

namespace hf {

constexpr int kWave = 64;            // CDNA wavefront width
constexpr int kMaxSelectBlocks = 2048;  // largest T_n the selection kernel ranks in LDS

typedef uint16_t bf16_t;  // storage type of a bfloat16 value

__device__ __forceinline__ float bf16_to_f32(bf16_t x) {
  return __uint_as_float(static_cast<uint32_t>(x) << 16);
}

// round-to-nearest-even; maps to v_cvt_pk_bf16_f32 on gfx950
__device__ __forceinline__ bf16_t f32_to_bf16(float f) {
  __bf16 b = static_cast<__bf16>(f);
  return __builtin_bit_cast(bf16_t, b);
}
// two of them, the first in the low half: one v_cvt_pk_bf16_f32 (joined from two scalars by shifts it is four instructions)
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const bf16x2 v = {static_cast<__bf16>(lo), static_cast<__bf16>(hi)};
  return __builtin_bit_cast(uint32_t, v);
}

template <typename T> struct Elem;
template <> struct Elem<float> {
  static constexpr int kPer16B = 4;
  __device__ static __forceinline__ float load(const float* p) { return *p; }
  __device__ static __forceinline__ void store(float* p, float v) { *p = v; }
};
template <> struct Elem<bf16_t> {
  static constexpr int kPer16B = 8;
  __device__ static __forceinline__ float load(const bf16_t* p) { return bf16_to_f32(*p); }
  __device__ static __forceinline__ void store(bf16_t* p, float v) { *p = f32_to_bf16(v); }
};

// 16-byte vector load of consecutive elements into fp32 registers
template <typename T> __device__ __forceinline__ void load16B(const T* p, float* out);
template <> __device__ __forceinline__ void load16B<float>(const float* p, float* out) {
  const float4 v = *reinterpret_cast<const float4*>(p);
  out[0] = v.x; out[1] = v.y; out[2] = v.z; out[3] = v.w;
}
template <> __device__ __forceinline__ void load16B<bf16_t>(const bf16_t* p, float* out) {
  const uint4 v = *reinterpret_cast<const uint4*>(p);
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    out[2 * i] = __uint_as_float(w[i] << 16);
    out[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
  }
}

// feature map of the linear branch (Eq. 2, 3): ReLU or elu(x)+1
__device__ __forceinline__ float phi_apply(float x, int kind) {
  if (kind == HF_PHI_RELU) return fmaxf(x, 0.0f);
  return x > 0.0f ? x + 1.0f : __expf(x);
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, kWave));
  return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}

// head_dim 128: one 32 x 32 tile of a head's state L[i][j] fp32 -> planes hi/lo, transposed: Lt[plane][j][i] bf16.  256 threads
__device__ __forceinline__ void state_planes_tile(const float* __restrict__ state, bf16_t* __restrict__ planes, int bh, int i0,
                                                  int j0, float (*tile)[33]) {
  constexpr int D = 128;
  const float* L = state + (size_t)bh * D * D;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
  for (int r = ty; r < 32; r += 8) tile[r][tx] = L[(size_t)(i0 + r) * D + j0 + tx];
  __syncthreads();
  bf16_t* hi = planes + (size_t)bh * 2 * D * D;
  bf16_t* lo = hi + D * D;
  for (int r = ty; r < 32; r += 8) {
    const float v = tile[tx][r];  // i = i0 + tx, j = j0 + r
    const bf16_t h = f32_to_bf16(v);
    hi[(size_t)(j0 + r) * D + i0 + tx] = h;
    lo[(size_t)(j0 + r) * D + i0 + tx] = f32_to_bf16(v - bf16_to_f32(h));
  }
}

// ---- host side -------------------------------------------------------------------------
void set_error(const char* fmt, ...);
int check_launch(const char* what);

// More than 64 KB of dynamic LDS has to be granted per kernel and device.  One object per kernel (static
// storage, zero-initialised); the grant is idempotent, so threads that race here at worst both ask for it.
struct LdsGrant {
  static constexpr int kDevices = 64;
  std::atomic<int> granted[kDevices];
};
int grant_lds(LdsGrant& g, const void* kernel, int bytes, const char* what);

// Per-call tag (48 bits) of the arrival counters that kernels keep in caller workspaces: a process-wide sequence
// from a random start, so that neither an earlier call's counters nor the uninitialised contents of a fresh
// workspace pass for this call's.  A counter word is (tag << 16) | count.
unsigned long long next_call_tag();

struct Dims {
  int B, H, D, BH;
  int n_q, n_kv, bq, bkv, t_m, t_n;
};

// tokens between the heads of K_win / V_win: the cache buffer's capacity, or the window length when packed
inline int kv_stride_of(const hf_config& c, int n_kv) { return c.kv_capacity > 0 ? c.kv_capacity : n_kv; }

// Launchers implemented in the .hip files.  All pointers are device pointers.
int launch_fill_zero(float* p, size_t n, hipStream_t s);
int launch_fold_linear(const hf_config& c, const float* state_in, const float* W, float* state_out, hipStream_t s);
int launch_absorb(const hf_config& c, float* state, const void* K, const void* V, int n, int head_stride,
                  const float* cosv, const float* sinv, void* workspace, size_t workspace_bytes,
                  hipStream_t s, void* planes_out = nullptr);
int launch_absorb_into(const hf_config& c, const float* state_in, float* state_out, const void* K, const void* V, int n,
                       int head_stride, const float* cosv, const float* sinv, void* workspace, size_t workspace_bytes,
                       hipStream_t s);
int launch_window_shift(const hf_config& c, void* K, void* V, int n_kv, int first, int n_evict, hipStream_t s);
size_t absorb_workspace_bytes(const hf_config& c, int n);
// pools every query block and the KV blocks [kv_first, kv_end); the other KV blocks keep what kbar_t holds
// state given (bf16, head_dim 128): its bf16 planes in the same launch
int launch_pool_both(const hf_config& c, const void* Q, int n_q, int t_m, const void* K, int n_kv, int t_n,
                     int kv_first, int kv_end, float* qbar, float* kbar_t, hipStream_t s, const float* state = nullptr,
                     void* planes = nullptr);
// both in one launch, where a head has little to pool and the workgroups are few
bool pool_select_supported(const hf_config& c, int t_m, int t_n, int kv_first, int kv_end);
int launch_pool_select(const hf_config& c, const void* Q, int n_q, int t_m, const void* K, int n_kv, int t_n, int kv_first,
                       int kv_end, int k, float* qbar, float* kbar_t, int32_t* idx, float* scores, hipStream_t s);
int launch_score_select(const hf_config& c, const float* qbar, const float* kbar_t, int t_m, int t_n,
                        int k, int32_t* idx, float* scores, hipStream_t s);
int launch_attn(const hf_config& c, const void* Q, int n_q, const void* K, const void* V, int n_kv,
                const int32_t* idx, int k, void* O_local, hipStream_t s);
// shapes whose attention kernel computes in fp32 and adds the history term itself
bool attn_wide_taken(const hf_config& c);
int launch_attn_wide_hist(const hf_config& c, const void* Q, const void* Q_hist, int n_q, const void* K, const void* V,
                          int n_kv, const int32_t* idx, int k, const float* state, const float* cosq, const float* sinq,
                          void* O, hipStream_t s);
int launch_readout_mfma(const hf_config& c, const void* Q, int n_q, const void* O_local, const float* state,
                        const float* cosq, const float* sinq, void* planes, void* O, hipStream_t s);
size_t readout_planes_bytes(const hf_config& c);  // scratch for the bf16 planes of the state
int launch_state_planes(const hf_config& c, const float* state, void* planes, hipStream_t s);
bool attn_mfma_fused_supported(const hf_config& c);
int launch_attn_mfma_fused(const hf_config& c, const void* Q, int n_q, const void* K, const void* V, int n_kv,
                           const int32_t* idx, int k, const void* planes, const float* zvec, const float* cosq,
                           const float* sinq, const void* Q_hist, void* O, hipStream_t s, float* lse2_out = nullptr,
                           void* olocal_out = nullptr,    // by-products for hf_hybrid_attn_bwd_saved, each optional
                           const float* kbar_t = nullptr, int32_t* idx_out = nullptr, float* scores_out = nullptr,
                           int pool_first = 0, int pool_end = 0,
                           const float* state = nullptr);   // L in place of planes (NULL then): rounded in the epilogue
// steps of small fp32 streams: selection, attention and, state_out given, Eq. 2 for another chunk into it, in one launch
bool attn_wide_step_supported(const hf_config& c, int n_q, int n_kv);
// against separate launches, k blocks a list; absorbs: the last step of the chunk absorbs beside its attention
bool attn_wide_step_pays(const hf_config& c, int n_q, int k, bool absorbs);
bool attn_wide_step_pools(const hf_config& c, int kv_first, int kv_end);
bool attn_wide_step_absorbs(const hf_config& c, int n_ev);
int launch_attn_wide_step(const hf_config& c, const void* Q, const void* Q_hist, int n_q, const void* K, const void* V, int n_kv, int k,
                          const float* state, const float* cosq, const float* sinq, float* kbar_t, int32_t* idx_out, int kv_first,
                          int kv_end, void* O, const void* K_ev, const void* V_ev, int n_ev, int ev_stride, const float* cos_ev,
                          const float* sin_ev, float* state_out, hipStream_t s);
bool attn_rounds_state_itself(const hf_config& c, int n_q, int n_kv, bool dense);
// kbar_t given (idx NULL): every workgroup selects its KV blocks itself (Eq. 4) and writes its list to idx_out; the blocks
// [pool_first, pool_end) it pools itself and stores in kbar_t (only where attn_pools_itself says so)
bool attn_pools_itself(const hf_config& c, int n_q, int t_n, int first, int end);
int launch_attn_mfma_select(const hf_config& c, const void* Q, int n_q, const void* K, const void* V, int n_kv, int k,
                            const float* kbar_t, int32_t* idx_out, float* scores_out, void* O_local, hipStream_t s,
                            int pool_first = 0, int pool_end = 0);
constexpr int kMaxFusedSelectBlocks = 1024;   // largest T_n the attention kernel ranks in its tile space
// the selecting launch with workgroups of their own that absorb n_ev tokens of another chunk (Eq. 2; ReLU, no
// rotation) into state_out / planes_out = state_in + their contribution; planes NULL: no history term in O
size_t step_absorb_workspace_bytes(const hf_config& c, int n_q, int n_ev);
int launch_attn_mfma_step(const hf_config& c, const void* Q, int n_q, const void* K, const void* V, int n_kv, int k,
                          const float* kbar_t, int32_t* idx_out, float* scores_out, const void* planes,
                          const float* zvec, const float* cosq, const float* sinq, const void* Q_hist, void* O,
                          const void* K_ev, const void* V_ev, int n_ev, int ev_stride, const float* state_in,
                          float* state_out, void* planes_out, void* workspace, hipStream_t s, int pool_first = 0,
                          int pool_end = 0);
int launch_attn_mfma_lse(const hf_config& c, const void* Q, int n_q, const void* K, const void* V, int n_kv,
                         const int32_t* idx, int k, void* O_local, float* lse2_out, hipStream_t s);
// backward pass (training algorithm): lse2 = per-row log2 of the softmax denominator in the scaled-logit domain
int launch_attn_wide_stats(const hf_config& c, const void* Q, int n_q, const void* K, const void* V, int n_kv,
                           const int32_t* idx, int k, const void* dO, float* lse2, float* dvec, hipStream_t s);
int launch_attn_mfma_stats(const hf_config& c, const void* Q, int n_q, const void* K, const void* V, int n_kv,
                           const int32_t* idx, int k, const void* dO, float* lse2, float* dvec, hipStream_t s);
bool bwd_mfma_supported(const hf_config& c);
size_t bwd_planes_bytes(const hf_config& c);
int launch_bwd_mfma(const hf_config& c, const void* Q, int n_q, const void* K, const void* V, int n_kv,
                    const int32_t* idx, int k, const void* dO, const float* lse2, const float* Dv,
                    const int32_t* inv_cnt, const int32_t* inv_list, const int32_t* order, const float* state,
                    const float* cosq, const float* sinq, const void* Q_hist, const void* planes, void* dQ, void* dQ_hist,
                    void* dK, void* dV, hipStream_t s);
// inverse lists, launch order of the dK/dV items, bf16 planes of the state, row dots: what is asked for, in one launch
constexpr int kOrderRec = 8;   // words per record of the launch order
int launch_bwd_prep(const hf_config& c, const int32_t* idx, int k, int t_m, int t_n, int32_t* inv_cnt, int32_t* inv_list,
                    int32_t* inv_slot, int32_t* order, int slabs, const float* state, void* planes, const void* A, const void* B, long long rows,
                    float* dots, hipStream_t s);
int launch_bwd_generic(const hf_config& c, const void* Q, const void* Q_hist, int n_q, const void* K, const void* V, int n_kv,
                       const int32_t* idx, int k, const void* dO, float* lse2, float* Dv, const int32_t* inv_cnt,
                       const int32_t* inv_list, const int32_t* inv_slot, const int32_t* order, float* scores, const float* state,
                       const float* zvec, const float* cosq, const float* sinq, void* dQ, void* dQ_hist, void* dK, void* dV, hipStream_t s);
size_t bwd_scores_room(const hf_config& c, int n_q, int k);                              // bytes that a workspace should have for scores
int bwd_scores_heads(const hf_config& c, int n_q, int n_kv, int k, size_t room);         // heads whose scores are stored at a time
int launch_rope_tables(const int32_t* frame_idx, int n_frames, int height, int width, int pairs_t, int pairs_h,
                       int pairs_w, double theta, int temporal_only, float* cosv, float* sinv, hipStream_t s);
int launch_rope_apply(const hf_config& c, const void* X, int n, const float* cosv, const float* sinv, void* Y,
                      hipStream_t s);
// the chunk's new keys rotated (tables NULL: copied) into the window at token `first`, the KV blocks they touch pooled
int launch_rope_append_pool(const hf_config& c, const void* X, int n_new, const float* cosv, const float* sinv, void* Kwin,
                            int first, int n_kv, float* kbar_t, hipStream_t s);

}  // namespace hf
