// Block-sparse window attention (Eq. 5) with the history term (Eq. 3, 6), shape-generic, fp32 arithmetic.
//
// Used for fp32 inputs (every product and sum in fp32, so the fp32-mode error bound holds) and for bf16 shapes that the
// bf16 matrix-core kernels do not cover.  Both products run on the fp32 matrix instruction (hf_f32_mfma.h), transposed as
// in the bf16 kernel, so that every statistic of a query row lives in the lanes of one column:
//   S^T (16 keys x 16 queries) = K (row form) x Q^T (row form)
//   O^T (D x 16 queries)      += V^T (column form) x P^T (= the C layout of S^T)
// A wavefront owns 16 NQ query rows; KS wavefronts share the same rows and split the list's 16-key tiles between them, and
// their partial results meet in LDS once, after the list.  The history term is added before that meeting, each of the KS
// wavefronts multiplying its share of the key features of L.
//
// Bound by the matrix pipes' fp32 rate (64 flops per cycle and SIMD): a tile's products take 1024 NQ cycles each at
// D = 128, next to 16 KB requested from the caches one phase ahead.
#include <stdlib.h>

#include <type_traits>

#include "hf_absorb_wide.h"
#include "hf_pool.h"

namespace hf {

namespace {

constexpr int kTile = 16;    // keys per tile

// What rides in the launch of a small stream's step: every workgroup selects the blocks of its rows itself, and workgroups of
// their own absorb another chunk into another state buffer.  Each of these is at the cost of a launch otherwise, and eight
// wavefronts share sixteen rows here instead of four.  A chunk, separate launches / this one: 2 heads of 64, 64 queries x 256 keys, blocks
// of 16, two steps 24.2 -> 20.3 us, 4 heads, 768 x 3072, half of the blocks, two steps 87 -> 63, 8 heads of 128, 512 x 1536, four steps
// 109 -> 102.  What such a launch takes is its longest chain: with the rows to pool requested together, a list by every wavefront for
// itself and the history term's operands requested under it, 2 heads of 64, 64 x 256, two steps 20.4 -> 18.8 us, 24 rings of such sizes
// 0.93 of the time in the mean.  (The same operands requested in front of the selection: 20.1, the rows to pool wait behind them; with
// the first keys: 1 us a step slower; the window's lines brought to the L2 under the Top-K: 19.8; the values with the first keys and a
// wavefront's blocks together: no difference.)
struct WideStep {
  float* kbar_t;          // [BH][D/4][T_n][4] pooled keys; those of the blocks [kv_first, kv_end) are formed here and stored
  int32_t* idx_out;       // [BH][T_m][k]
  int kv_first, kv_end;
  const void *K_ev, *V_ev;
  int n_ev, ev_stride;
  const float *cos_ev, *sin_ev, *state_in;
  float* state_out;
  int role_blocks, BH;    // the first workgroup ids (a multiple of eight) absorb
};
constexpr int kStepWaves = 8, kStepOwn = 16, kStepBlocks = 256;   // wavefronts; most blocks pooled in the launch, in the window

// Eq. 4 and the Top-K for one query block by eight wavefronts; sums in the order of pool_kernel and select_rows, so that the list
// is theirs.  The list is left at sel; scratch: D + 9 t_pad + 16 D floats at smem.  `under` runs behind the scores: what it requests
// arrives under the Top-K (in front, the rows to pool wait behind it).
template <typename T, int D, typename Under>
__device__ __forceinline__ void select_block(float* smem, int* sel, const T* Qh, int q0, int q1, const T* Kh, int n_kv, int bkv,
                                             int t_n, int k, float* kbar_head, int kv_first, int kv_end, bool store,
                                             int32_t* idx_row, Under under) {
  using P = Pool<T, D>;
  constexpr int E = P::E, CW = D / 32;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int t_pad = (t_n + 3) & ~3;
  float* sq = smem;
  float* part = sq + D;                 // [8][t_pad]
  float* sc = part + kStepWaves * t_pad;
  float* fresh = sc + t_pad;            // [kStepOwn][D]
  __shared__ unsigned long long masks[kStepWaves];
  const float4* kt = reinterpret_cast<const float4*>(kbar_head) + (size_t)wave * CW * t_n;
  float4 kv[4][CW];                     // (requested first: what was pooled before is on its way while the rest is pooled)
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (64 * u < t_n) {                 // uniform
      const int j = min(lane + 64 * u, t_n - 1);
#pragma unroll
      for (int c = 0; c < CW; ++c) kv[u][c] = kt[(size_t)c * t_n + j];
    }
  const int sub = lane / P::LPR, col = (lane % P::LPR) * E;
  // a wavefront's items are every eighth block to pool, the last one the query block
  const int items = kv_end - kv_first + 1;
  auto rows_of = [&](int it, bool& is_q, int& r0, int& r1) {
    is_q = it == items - 1;
    r0 = is_q ? q0 : (kv_first + it) * bkv;
    r1 = is_q ? q1 : min(n_kv, r0 + bkv);
  };
  auto keep_mean = [&](int it, bool is_q, const float (&acc)[E]) {
    const int blk = kv_first + it;
    if (sub == 0) {
#pragma unroll
      for (int e = 0; e < E; e += 4) {
        const float4 v = make_float4(acc[e], acc[e + 1], acc[e + 2], acc[e + 3]);
        *reinterpret_cast<float4*>((is_q ? sq : fresh + it * D) + col + e) = v;
        if (!is_q && store) reinterpret_cast<float4*>(kbar_head)[(size_t)((col + e) / 4) * t_n + blk] = v;
      }
    }
  };
  if (max(bkv, q1 - q0) <= P::kFew) {   // (uniform) short blocks: all of a wavefront's rows are requested before the first mean
    constexpr int MAXI = (kStepOwn + 1 + kStepWaves - 1) / kStepWaves;
    float v[MAXI][8][E];
#pragma unroll
    for (int i = 0; i < MAXI; ++i)
      if (wave + kStepWaves * i < items) {   // uniform
        bool is_q; int r0, r1;
        rows_of(wave + kStepWaves * i, is_q, r0, r1);
        P::request((is_q ? Qh : Kh) + col, r0, r1, sub, v[i]);
      }
#pragma unroll
    for (int i = 0; i < MAXI; ++i)
      if (wave + kStepWaves * i < items) {
        bool is_q; int r0, r1;
        float acc[E];
        rows_of(wave + kStepWaves * i, is_q, r0, r1);
        P::mean_of(v[i], r0, r1, sub, acc);
        keep_mean(wave + kStepWaves * i, is_q, acc);
      }
  } else {
    for (int it = wave; it < items; it += kStepWaves) {   // uniform
      bool is_q; int r0, r1;
      float acc[E];
      rows_of(it, is_q, r0, r1);
      P::template mean<true>((is_q ? Qh : Kh) + col, r0, r1, sub, acc);
      keep_mean(it, is_q, acc);
    }
  }
  if (tid < t_pad - t_n) sc[t_n + tid] = -INFINITY;   // never outranks a block
  __syncthreads();
  const float4* q4 = reinterpret_cast<const float4*>(sq) + wave * CW;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int j = lane + 64 * u;
    if (j < t_n) {
      const bool mine = j >= kv_first && j < kv_end;
      float a = 0.0f;
#pragma unroll
      for (int c = 0; c < CW; ++c) {
        const float4 q = q4[c], x = mine ? *reinterpret_cast<const float4*>(fresh + (j - kv_first) * D + 4 * (wave * CW + c)) : kv[u][c];
        a = fmaf(q.x, x.x, a); a = fmaf(q.y, x.y, a); a = fmaf(q.z, x.z, a); a = fmaf(q.w, x.w, a);
      }
      part[wave * t_pad + j] = a;
    }
  }
  under();
  __syncthreads();
  auto score_of = [&](int j) {
    const float* x = part + j;
    return ((x[0] + x[t_pad]) + (x[2 * t_pad] + x[3 * t_pad])) + ((x[4 * t_pad] + x[5 * t_pad]) + (x[6 * t_pad] + x[7 * t_pad]));
  };
  if (t_n <= 64) {
    // every wavefront for itself, a lane a block, by the same comparisons: all write the same list, and nobody waits for anybody
    const float mine = score_of(min(lane, t_n - 1));
    int rank = 0;
    for (int o = 0; o < t_n; ++o) {
      const float v = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(mine), o));
      rank += (v > mine || (v == mine && o < lane)) ? 1 : 0;
    }
    const bool keep = lane < t_n && rank < k;
    const int pos = __popcll(__ballot(keep) & ((1ull << lane) - 1ull));
    if (keep && pos < k) {
      sel[pos] = lane;
      if (idx_row && wave == 0) idx_row[pos] = lane;
    }
    return;   // (what the workgroup leaves at smem next lies behind this scratch or a barrier)
  }
  if (tid < t_n) {
    sc[tid] = score_of(tid);
  }
  __syncthreads();
  // a block's rank among the row's scores, equal ones by index; the list by ballots
  bool keep = false;
  if (tid < t_n) {
    const float mine = sc[tid];
    int rank = 0;
    for (int o = 0; o < t_pad; o += 4) {
      const float4 v = *reinterpret_cast<const float4*>(sc + o);
      rank += (v.x > mine || (v.x == mine && o < tid)) ? 1 : 0;
      rank += (v.y > mine || (v.y == mine && o + 1 < tid)) ? 1 : 0;
      rank += (v.z > mine || (v.z == mine && o + 2 < tid)) ? 1 : 0;
      rank += (v.w > mine || (v.w == mine && o + 3 < tid)) ? 1 : 0;
    }
    keep = rank < k;
  }
  const unsigned long long m = __ballot(keep);
  if (lane == 0) masks[wave] = m;
  __syncthreads();
  int pos = __popcll(m & ((1ull << lane) - 1ull));
  for (int w = 0; w < wave; ++w) pos += __popcll(masks[w]);
  if (keep && pos < k) {
    sel[pos] = tid;
    if (idx_row) idx_row[pos] = tid;
  }
  __syncthreads();
}

// phi of a history term's queries (one uniform choice of the feature map: a branch for every feature kept the loads apart)
template <int NQ, int C>
__device__ __forceinline__ void apply_phi(f32x4 (&ph)[NQ][C], int phi_kind) {
  if (phi_kind == HF_PHI_RELU) {
#pragma unroll
    for (int n = 0; n < NQ; ++n)
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) ph[n][c][e] = phi_apply(ph[n][c][e], HF_PHI_RELU);
  } else {
#pragma unroll
    for (int n = 0; n < NQ; ++n)
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) ph[n][c][e] = phi_apply(ph[n][c][e], HF_PHI_ELU1);
  }
}
// R f of a row's features
template <int D>
__device__ __forceinline__ void rotate_features(f32x4 (&ph)[D / 16], const WideHist& hist, size_t qrow, int g) {
#pragma unroll
  for (int c = 0; c < D / 16; ++c) {
    const size_t at = qrow * (D / 2) + 8 * c + 2 * g;
    const float2 cs = *reinterpret_cast<const float2*>(hist.cosq + at), sn = *reinterpret_cast<const float2*>(hist.sinq + at);
    ph[c] = rotate4(ph[c], cs.x, sn.x, cs.y, sn.y);
  }
}

template <typename T, int D, int NQ, int KS, int NWV, bool kSel>
__global__ __launch_bounds__(64 * NWV, 2) void attn_wide_kernel(const T* __restrict__ Q, const T* __restrict__ K,
                                                           const T* __restrict__ V, const int32_t* __restrict__ idx, int k,
                                                           int n_q, int n_kv, int kv_stride, int bq, int bkv, int t_m,
                                                           int t_n, int chunks, int per_xcd, int total, float scale_log2e,
                                                           WideHist hist, WideStep step, T* __restrict__ O) {
  constexpr int WR = NWV / KS;           // wavefronts along the rows
  constexpr int ROWS = WR * 16 * NQ;     // query rows of a workgroup
  constexpr int C = D / 16;              // row-form pieces of a token
  constexpr int F = D / 64;              // column-form pieces of a token
  constexpr int OST = D + 4;             // floats per row of a partial result in LDS (breaks the banks' period)
  extern __shared__ __attribute__((aligned(16))) float smem[];
  if constexpr (kSel) {
    static_assert(5 * sizeof(void*) + 11 * sizeof(int) + sizeof(WideHist) + sizeof(WideStep) >= 196, "four lines of arguments");
    warm_arguments<4>();
  }
  // one contiguous run of (head, query block, chunk of rows) per XCD: its L2 then holds the keys of few heads
  int wg = blockIdx.x;
  if constexpr (kSel) {
    if (wg < step.role_blocks) {
      constexpr int TILES = (D / 32) * (D / 32);
      if (wg < step.BH * TILES)
        absorb_tile<T, D>(smem, wg % TILES, 0, wg / TILES, step.state_in, step.state_out, static_cast<const T*>(step.K_ev),
                          static_cast<const T*>(step.V_ev), step.n_ev, step.ev_stride, step.n_ev, step.cos_ev, step.sin_ev,
                          hist.phi_kind, step.BH, 1);
      return;
    }
    wg -= step.role_blocks;
  }
  const int item = (wg & 7) * per_xcd + (wg >> 3);
  if ((wg >> 3) >= per_xcd || item >= total) return;
  const int bh = item / (t_m * chunks), in_head = item - bh * t_m * chunks;
  const int qb = in_head / chunks, chunk = in_head - qb * chunks;
  const int row0 = qb * bq + chunk * ROWS;
  const int q_end = min(n_q, (qb + 1) * bq);
  if (row0 >= q_end) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  const int wr = wave / KS, kz = wave % KS;
  const T* Kh = K + (size_t)bh * kv_stride * D;  // heads of a cache buffer are kv_stride tokens apart
  const T* Vh = V + (size_t)bh * kv_stride * D;
  const int32_t* row_idx = idx ? idx + ((size_t)bh * t_m + qb) * k : nullptr;
  const int nsel = kSel || idx ? k : t_n;
  const int subs = (bkv + kTile - 1) / kTile;
  const int ntiles = nsel * subs;
  int* const sel = reinterpret_cast<int*>(smem + KS * ROWS * OST + ROWS * KS * 2);   // kSel: the list, behind everything else

  // rows past the block's end are computed on clamped addresses and never written
  int row[NQ];
  f32x4 qf[NQ][C];
  if constexpr (!kSel) {
#pragma unroll
    for (int n = 0; n < NQ; ++n) {
      row[n] = row0 + 16 * (wr * NQ + n) + l16;
      const T* qp = Q + ((size_t)bh * n_q + min(row[n], n_q - 1)) * D + 4 * g;
#pragma unroll
      for (int c = 0; c < C; ++c) qf[n][c] = load4<T>(qp + 16 * c) * scale_log2e;
    }
  }
  // Selecting, the queries are requested under the selection, at D = 64 with the history term's operands: its features and denominator
  // are formed in front of the loop then, while the first keys travel (elsewhere the registers are the selection's and the loop's).
  // What the other instances do stands apart from it, so that they are compiled as if there were no selection.
  constexpr bool kHistEarly = kSel && D == 64;
  f32x4 ph_early[kHistEarly ? NQ : 1][C], zz[kHistEarly ? C : 1];
  float den_early[kHistEarly ? NQ : 1];
  if constexpr (kSel) {
    float warm_l = 0.0f;
    auto under = [&]() {
#pragma unroll
      for (int n = 0; n < NQ; ++n) {
        row[n] = row0 + 16 * (wr * NQ + n) + l16;
        const T* qp = Q + ((size_t)bh * n_q + min(row[n], n_q - 1)) * D + 4 * g;
#pragma unroll
        for (int c = 0; c < C; ++c) qf[n][c] = load4<T>(qp + 16 * c) * scale_log2e;
      }
      if (hist.L) {
        // (the state, D^2 / 32 lines of 128 bytes, is brought to the L2 ahead of its use)
        static_assert(!kSel || D * D / 32 <= 64 * NWV, "a line a thread");
        warm_l = hist.L[(size_t)bh * D * D + 32 * (threadIdx.x & (D * D / 32 - 1))];
        if constexpr (kHistEarly) {
          const T* qh = static_cast<const T*>(hist.q_hist);
          const float* z = hist.z + (size_t)bh * D + 4 * g;
#pragma unroll
          for (int n = 0; n < NQ; ++n)
#pragma unroll
            for (int c = 0; c < C; ++c) ph_early[n][c] = load4<T>(qh + ((size_t)bh * n_q + min(row[n], n_q - 1)) * D + 16 * c + 4 * g);
#pragma unroll
          for (int c = 0; c < C; ++c) zz[c] = *reinterpret_cast<const f32x4*>(z + 16 * c);
        }
      }
    };
    select_block<T, D>(smem, sel, Q + (size_t)bh * n_q * D, qb * bq, q_end, Kh, n_kv, bkv, t_n, k,
                       step.kbar_t + (size_t)bh * D * t_n, step.kv_first, step.kv_end, in_head == 0,
                       chunk == 0 ? step.idx_out + ((size_t)bh * t_m + qb) * k : nullptr, under);
    asm volatile("" :: "v"(warm_l));
  }

  f32x4 o[NQ][F][4];
  float m[NQ], l[NQ];
#pragma unroll
  for (int n = 0; n < NQ; ++n) {
    m[n] = -INFINITY;
    l[n] = 0.0f;
#pragma unroll
    for (int f = 0; f < F; ++f)
#pragma unroll
      for (int e = 0; e < 4; ++e) o[n][f][e] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  }

  // tile t of the list: first key and number of real keys (0: past the list, an index out of range, or an empty part of a
  // short block); the rows behind them read as zeros and their scores are -inf
  auto tile_at = [&](int t, int& first, int& cnt) {
    const int s = t / subs, sub = t - s * subs;
    const int jb = kSel ? __builtin_amdgcn_readfirstlane(sel[min(s, nsel - 1)]) : row_idx ? row_idx[min(s, nsel - 1)] : s;
    const int st = jb * bkv + kTile * sub;
    const bool ok = s < nsel && (unsigned)jb < (unsigned)t_n;
    const int n = ok ? min(kTile, min(n_kv, (jb + 1) * bkv) - st) : 0;
    cnt = n > 0 ? n : 0;
    first = n > 0 ? st : 0;
  };
  Piece<T> kp[C], vp[4][F];
  constexpr int B = sizeof(T);
  int k_at = (l16 * D + 4 * g) * B, v_at = (4 * g * D + 4 * l16) * B;
  auto load_k = [&](int first, int cnt) {
    const __amdgpu_buffer_rsrc_t rows = tile_rows<T, D>(Kh, first, cnt);
#pragma unroll
    for (int c = 0; c < C; ++c) kp[c].load(rows, k_at + 16 * c * B);
  };
  auto load_v = [&](int first, int cnt) {
    const __amdgpu_buffer_rsrc_t rows = tile_rows<T, D>(Vh, first, cnt);
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int f = 0; f < F; ++f) vp[r][f].load(rows, v_at + (r * D + 64 * f) * B);
  };

  // One tile ahead in every direction: trip t forms the scores of tile t + 1 next to the exponentials of tile t (the matrix
  // instructions of the one hide the vector work of the other, also for a wavefront that is alone on its SIMD), then
  // accumulates tile t.  Its keys were requested before tile t - 1 was accumulated, its values behind that.
  f32x4 sc[NQ];
  auto scores = [&]() {
    f32x4 s[NQ][2];
#pragma unroll
    for (int n = 0; n < NQ; ++n) s[n][0] = s[n][1] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const f32x4 a = kp[c].get();
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int n = 0; n < NQ; ++n) s[n][e & 1] = mfma_f32(a[e], qf[n][c][e], s[n][e & 1]);
    }
#pragma unroll
    for (int n = 0; n < NQ; ++n) sc[n] = s[n][0] + s[n][1];
  };
  // missing keys of the tile to -inf, its maximum into the reference m; what was accumulated under a smaller reference is
  // scaled (rarely: only once the maximum has grown by more than 2^8, any reference is exact in floating point)
  auto maxima = [&](int cnt) {
    bool grow = false;
    float mx[NQ];
#pragma unroll
    for (int n = 0; n < NQ; ++n) {
#pragma unroll
      for (int r = 0; r < 4; ++r) sc[n][r] = 4 * g + r < cnt ? sc[n][r] : -INFINITY;
      mx[n] = column_max(fmaxf(fmaxf(sc[n][0], sc[n][1]), fmaxf(sc[n][2], sc[n][3])));
      grow |= mx[n] > m[n] + 8.0f;
    }
    if (__any(grow)) {
#pragma unroll
      for (int n = 0; n < NQ; ++n) {
        const float m_new = fmaxf(m[n], mx[n]);
        const float alpha = exp2f(m[n] - (m_new == -INFINITY ? 0.0f : m_new));
        m[n] = m_new;
        l[n] *= alpha;
#pragma unroll
        for (int f = 0; f < F; ++f)
#pragma unroll
          for (int e = 0; e < 4; ++e) o[n][f][e] *= alpha;
      }
    }
  };
  f32x4 p[NQ];
  auto weights = [&]() {
#pragma unroll
    for (int n = 0; n < NQ; ++n) {
      const float m_use = m[n] == -INFINITY ? 0.0f : m[n];   // nothing seen yet: keep the exponents finite
#pragma unroll
      for (int r = 0; r < 4; ++r) p[n][r] = __builtin_amdgcn_exp2f(sc[n][r] - m_use);
      l[n] += (p[n][0] + p[n][1]) + (p[n][2] + p[n][3]);     // this lane's keys only; summed at the end
    }
  };
  auto accumulate = [&]() {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int f = 0; f < F; ++f) {
        const f32x4 a = vp[r][f].get();
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int n = 0; n < NQ; ++n) o[n][f][e] = mfma_f32(a[e], p[n][r], o[n][f][e]);
      }
  };
  int first_v, cnt, first_k, cnt_k;
  tile_at(kz, first_v, cnt);
  load_k(first_v, cnt);
  tile_at(kz + KS, first_k, cnt_k);
  if constexpr (kHistEarly) {
    if (hist.L) {
      apply_phi(ph_early, hist.phi_kind);
#pragma unroll
      for (int n = 0; n < NQ; ++n) {
        float acc = 0.0f;
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc = fmaf(ph_early[n][c][e], zz[c][e], acc);
        if (hist.cosq) rotate_features<D>(ph_early[n], hist, (size_t)min(row[n], n_q - 1), g);
        den_early[n] = hist.z_scale * column_sum(acc) + hist.eps;
      }
    }
  }
  scores();
  load_k(first_k, cnt_k);
  __builtin_amdgcn_sched_barrier(0);   // (requests are awaited in order: values behind keys, here as in the loop)
  load_v(first_v, cnt);
  __builtin_amdgcn_sched_barrier(0);
  maxima(cnt);
  for (int t = kz; t < ntiles; t += KS) {
    asm volatile("" : "+v"(k_at), "+v"(v_at));   // (opaque here, or their sums leave the loop as registers instead of immediates)
    first_v = first_k;
    cnt = cnt_k;
    tile_at(t + 2 * KS, first_k, cnt_k);
    weights();
    scores();
#pragma unroll
    for (int u = 0; u < 4 * C * NQ; ++u) {   // one matrix instruction, then the vector work it hides
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
    }
    load_k(first_k, cnt_k);
    __builtin_amdgcn_sched_barrier(0);
    accumulate();
    load_v(first_v, cnt);
    __builtin_amdgcn_sched_barrier(0);
    maxima(cnt);
  }

  // (kSel: a wavefront takes at most one run of 16 key features of the history term; its part of L travels under the meeting)
  f32x4 lv_of[kSel ? 4 : 1][kSel ? F : 1];
  if constexpr (kSel) {
    static_assert(C <= KS, "one run a wavefront");
    if (hist.L && kz < C) {   // uniform
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int f = 0; f < F; ++f)
          lv_of[r][f] = *reinterpret_cast<const f32x4*>(hist.L + (size_t)bh * D * D + 4 * l16 + (size_t)(16 * kz + 4 * g + r) * D + 64 * f);
    }
  }
  // ---- weights of the KS parts of a row: w = 2^(m_part - m) / l
  float w[NQ];
#pragma unroll
  for (int n = 0; n < NQ; ++n) l[n] = column_sum(l[n]);
  float* parts = smem + (KS > 1 ? KS * (ROWS / WR) * WR * OST : 0);   // [ROWS][KS][2], behind the partial results
  if (KS > 1) {
#pragma unroll
    for (int n = 0; n < NQ; ++n)
      if (g == 0) {
        float* q = parts + ((16 * (wr * NQ + n) + l16) * KS + kz) * 2;
        q[0] = m[n];
        q[1] = l[n];
      }
    __syncthreads();
#pragma unroll
    for (int n = 0; n < NQ; ++n) {
      const float* q = parts + (16 * (wr * NQ + n) + l16) * KS * 2;
      float mt = -INFINITY, lt = 0.0f;
#pragma unroll
      for (int u = 0; u < KS; ++u) mt = fmaxf(mt, q[2 * u]);
      const float m_use = mt == -INFINITY ? 0.0f : mt;
#pragma unroll
      for (int u = 0; u < KS; ++u) lt = fmaf(q[2 * u + 1], exp2f(q[2 * u] - m_use), lt);
      w[n] = exp2f(m[n] - m_use);
      m[n] = mt;
      l[n] = lt;
    }
  } else {
#pragma unroll
    for (int n = 0; n < NQ; ++n) w[n] = 1.0f;
  }
#pragma unroll
  for (int n = 0; n < NQ; ++n) w[n] = l[n] > 0.0f ? w[n] / l[n] : 0.0f;   // a row without a single real key: O_local = 0

  float den[NQ];
#pragma unroll
  for (int n = 0; n < NQ; ++n) den[n] = 1.0f;
  if (hist.L) {
    // ---- O += R(phi(q)) L / (z_scale phi(q).z + eps) (Eq. 3, 6): O_local is scaled by the denominator, the products add
    // the numerator to the same accumulators (L in column form, its key features in the place of tokens), one division
    // at the end.  Each of the KS wavefronts takes every KS-th run of 16 key features.
    const float* L = hist.L + (size_t)bh * D * D + 4 * l16;
    const float* z = hist.z + (size_t)bh * D + 4 * g;
    const T* qh = static_cast<const T*>(hist.q_hist);
    f32x4 ph[NQ][C];
    if constexpr (!kHistEarly) {   // (all loads first)
#pragma unroll
      for (int n = 0; n < NQ; ++n)
#pragma unroll
        for (int c = 0; c < C; ++c) ph[n][c] = load4<T>(qh + ((size_t)bh * n_q + min(row[n], n_q - 1)) * D + 16 * c + 4 * g);
      apply_phi(ph, hist.phi_kind);
    }
#pragma unroll
    for (int n = 0; n < NQ; ++n) {
      if constexpr (kHistEarly) {
#pragma unroll
        for (int c = 0; c < C; ++c) ph[n][c] = ph_early[n][c];
        den[n] = den_early[n];
      } else {
        const size_t qrow = (size_t)min(row[n], n_q - 1);
        float acc = 0.0f;
#pragma unroll
        for (int c = 0; c < C; ++c) {
          const f32x4 zc = *reinterpret_cast<const f32x4*>(z + 16 * c);
#pragma unroll
          for (int e = 0; e < 4; ++e) acc = fmaf(ph[n][c][e], zc[e], acc);
        }
        if (hist.cosq) rotate_features<D>(ph[n], hist, qrow, g);
        den[n] = hist.z_scale * column_sum(acc) + hist.eps;
      }
      w[n] *= den[n];
#pragma unroll
      for (int f = 0; f < F; ++f)
#pragma unroll
        for (int e = 0; e < 4; ++e) o[n][f][e] *= w[n];
    }
#pragma unroll
    for (int c = 0; c < C; ++c) {
      if (c % KS != kz) continue;   // uniform
      f32x4 lv[4][F];
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int f = 0; f < F; ++f) {
          if constexpr (kSel) lv[r][f] = lv_of[r][f];
          else lv[r][f] = *reinterpret_cast<const f32x4*>(L + (size_t)(16 * c + 4 * g + r) * D + 64 * f);
        }
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int f = 0; f < F; ++f)
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int n = 0; n < NQ; ++n) o[n][f][e] = mfma_f32(lv[r][f][e], ph[n][c][r], o[n][f][e]);
    }
#pragma unroll
    for (int n = 0; n < NQ; ++n) den[n] = 1.0f / den[n];
  } else {
#pragma unroll
    for (int n = 0; n < NQ; ++n)
#pragma unroll
      for (int f = 0; f < F; ++f)
#pragma unroll
        for (int e = 0; e < 4; ++e) o[n][f][e] *= w[n];
  }

  if (hist.lse2) {
    // ---- statistics for the backward pass: log2 of the sum of 2^(scaled logit), and D = dO . O_local from the unrounded
    // output.  The KS parts of O_local are summed as scalars.
    const T* dO = static_cast<const T*>(hist.d_out);
#pragma unroll
    for (int n = 0; n < NQ; ++n) {
      float acc = 0.0f;
      const T* gp = dO + ((size_t)bh * n_q + min(row[n], n_q - 1)) * D + 16 * g;
#pragma unroll
      for (int f = 0; f < F; ++f)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const f32x4 x = load4<T>(gp + 64 * f + 4 * r);
#pragma unroll
          for (int e = 0; e < 4; ++e) acc = fmaf(o[n][f][e][r], x[e], acc);
        }
      acc = column_sum(acc);
      if (KS > 1) {
        float* q = smem + (16 * (wr * NQ + n) + l16) * KS;   // (the partial results' place is not used here)
        if (g == 0) q[kz] = acc;
        __syncthreads();
        acc = 0.0f;
#pragma unroll
        for (int u = 0; u < KS; ++u) acc += q[u];
      }
      if (g == 0 && kz == 0 && row[n] < q_end) {
        hist.lse2[(size_t)bh * n_q + row[n]] = l[n] > 0.0f ? m[n] + log2f(l[n]) : INFINITY;  // no real key: P = 0
        hist.dvec[(size_t)bh * n_q + row[n]] = acc;
      }
    }
    return;
  }

  if (KS == 1) {
#pragma unroll
    for (int n = 0; n < NQ; ++n)
      if (row[n] < q_end) {
        T* op = O + ((size_t)bh * n_q + row[n]) * D + 16 * g;
#pragma unroll
        for (int f = 0; f < F; ++f)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            store4<T>(op + 64 * f + 4 * r,
                      f32x4{o[n][f][0][r], o[n][f][1][r], o[n][f][2][r], o[n][f][3][r]} * den[n]);
      }
    return;
  }
  // ---- the KS parts of a row meet in LDS; the workgroup's threads add them and store whole rows
#pragma unroll
  for (int n = 0; n < NQ; ++n) {
    float* dst = smem + ((size_t)kz * ROWS + 16 * (wr * NQ + n) + l16) * OST + 16 * g;
#pragma unroll
    for (int f = 0; f < F; ++f)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        *reinterpret_cast<f32x4*>(dst + 64 * f + 4 * r) =
            f32x4{o[n][f][0][r], o[n][f][1][r], o[n][f][2][r], o[n][f][3][r]} * den[n];
  }
  __syncthreads();
  for (int e = threadIdx.x; e < ROWS * (D / 4); e += 64 * NWV) {
    const int rr = e / (D / 4), c4 = e - rr * (D / 4);
    if (row0 + rr >= q_end) continue;
    f32x4 v = *reinterpret_cast<const f32x4*>(smem + (size_t)rr * OST + 4 * c4);
#pragma unroll
    for (int u = 1; u < KS; ++u) v += *reinterpret_cast<const f32x4*>(smem + ((size_t)u * ROWS + rr) * OST + 4 * c4);
    store4<T>(O + ((size_t)bh * n_q + row0 + rr) * D + 4 * c4, v);
  }
}

template <typename T, int D, int NQ, int KS>
int launch_wide(const hf_config& c, const void* Q, int n_q, const void* K, const void* V, int n_kv, const int32_t* idx,
                int k, void* O, const WideHist& hist, hipStream_t s) {
  constexpr int ROWS = 16 * NQ * 4 / KS;
  const int BH = c.batch * c.heads;
  const int t_m = (n_q + c.block_q - 1) / c.block_q, t_n = (n_kv + c.block_kv - 1) / c.block_kv;
  const int chunks = (c.block_q + ROWS - 1) / ROWS;
  const long long total = (long long)BH * t_m * chunks;
  if (total > (1ll << 30)) { set_error("too many query blocks"); return HF_ERR_SHAPE; }
  const int per_xcd = (int)((total + 7) / 8);
  const float scale = c.softmax_scale > 0.0f ? c.softmax_scale : 1.0f / sqrtf((float)c.head_dim);
  const size_t lds = KS > 1 ? ((size_t)KS * ROWS * (D + 4) + (size_t)ROWS * KS * 2) * sizeof(float) : 0;
  auto kern = attn_wide_kernel<T, D, NQ, KS, 4, false>;
  if (lds > 64 * 1024) {
    static LdsGrant grant;   // (one per instantiation, i.e. per kernel)
    const int rc = grant_lds(grant, reinterpret_cast<const void*>(kern), (int)lds, "the fp32 attention kernel");
    if (rc != HF_OK) return rc;
  }
  hipLaunchKernelGGL(kern, dim3(8 * per_xcd), dim3(256), lds, s, static_cast<const T*>(Q), static_cast<const T*>(K),
                     static_cast<const T*>(V), idx, k, n_q, n_kv, kv_stride_of(c, n_kv), c.block_q, c.block_kv, t_m, t_n,
                     chunks, per_xcd, (int)total, scale * 1.4426950408889634f, hist, WideStep{}, static_cast<T*>(O));
  return check_launch("hf_hybrid_attn_fwd(attention)");
}

// the step of a small stream: sixteen rows a workgroup, eight wavefronts that share them
template <int D>
int launch_wide_step_d(const hf_config& c, const void* Q, int n_q, const void* K, const void* V, int n_kv, int k, void* O,
                       const WideHist& hist, WideStep step, hipStream_t s) {
  constexpr int ROWS = 16, KS = kStepWaves;
  const int BH = c.batch * c.heads;
  const int t_m = (n_q + c.block_q - 1) / c.block_q, t_n = (n_kv + c.block_kv - 1) / c.block_kv;
  const int chunks = (c.block_q + ROWS - 1) / ROWS;
  const long long total = (long long)BH * t_m * chunks;
  const int per_xcd = (int)((total + 7) / 8);
  const float scale = c.softmax_scale > 0.0f ? c.softmax_scale : 1.0f / sqrtf((float)c.head_dim);
  constexpr int kFloats = KS * ROWS * (D + 4) + ROWS * KS * 2;
  constexpr int lds = kFloats * (int)sizeof(float) + kStepBlocks * (int)sizeof(int);
  static_assert(kFloats >= D + 9 * kStepBlocks + kStepOwn * D && lds >= kAbsorbLds, "selection and absorb use the same space");
  step.BH = BH;
  step.role_blocks = step.state_out ? (BH * (D / 32) * (D / 32) + 7) & ~7 : 0;
  auto kern = attn_wide_kernel<float, D, 1, KS, kStepWaves, true>;
  if (lds > 64 * 1024) {
    static LdsGrant grant;
    const int rc = grant_lds(grant, reinterpret_cast<const void*>(kern), lds, "the fp32 step kernel");
    if (rc != HF_OK) return rc;
  }
  hipLaunchKernelGGL(kern, dim3(8 * per_xcd + step.role_blocks), dim3(64 * kStepWaves), lds, s, static_cast<const float*>(Q),
                     static_cast<const float*>(K), static_cast<const float*>(V), nullptr, k, n_q, n_kv, kv_stride_of(c, n_kv),
                     c.block_q, c.block_kv, t_m, t_n, chunks, per_xcd, (int)total, scale * 1.4426950408889634f, hist, step,
                     static_cast<float*>(O));
  return check_launch("hf_ring_step(selection, attention)");
}

// ---- fp32 storage, block_q and block_kv multiples of 32, few rows: tiles of 32 keys x 32 queries on the 32 x 32 x 2 instruction.
// A workgroup owns 32 query rows of a block; its four wavefronts take every fourth tile of the list and meet in LDS once,
// at the end.  A trip forms the scores of the wavefront's next tile next to the exponentials of the current one and then
// accumulates the current one; every 16-byte piece is requested one such phase (4096 cycles at D = 128) before its use,
// into the registers of a piece that has just been used.  Tile addresses are scalar (the tile's first row moves into the
// buffer descriptor, whose end is the tile's last real row: what lies behind reads as zero).
// Measured at 832x480 in fp32 (12 heads of 128, 4680 x 9360, k = 37 of 147 blocks of 64; selection included): 4.84 ms with
// one key per lane and FMA arithmetic, 0.67 ms with the 16 x 16 tiles below, 0.61 ms (115 of the 154 TFLOP/s the
// instruction sustains) with this kernel: the pipes are 86 % busy while a compute unit has work, and the last of 3.5 rounds
// of workgroups leaves an eighth of the chip idle.  Launches of more than 128 blocks of 64 rows are faster still in bf16 products
// (hf_attn_f32.hip).
template <int D>
__global__ __launch_bounds__(256, 2) void attn_wide32_kernel(const float* __restrict__ Q, const float* __restrict__ K,
                                                             const float* __restrict__ V, const int32_t* __restrict__ idx,
                                                             int k, int n_q, int n_kv, int kv_stride, int bq, int bkv,
                                                             int t_m, int t_n, int per_xcd, int total, float scale_log2e,
                                                             WideHist hist, float* __restrict__ O) {
  constexpr int KS = 4;                  // wavefronts that share the rows
  constexpr int C = D / 8;               // row-form pieces of a token
  constexpr int E = D / 32;              // 32-row operands of a column-form piece (features E i + e)
  constexpr int OST = D + 4;             // floats per row of a partial result in LDS
  constexpr int ROWB = D * 4;
  typedef float vpiece __attribute__((ext_vector_type(E)));
  __shared__ __attribute__((aligned(16))) float part[KS][32][OST];
  __shared__ float stat[32][KS][2];
  const int item = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per_xcd || item >= total) return;
  const int chunks = bq >> 5;
  const int bh = item / (t_m * chunks), in_head = item - bh * t_m * chunks;
  const int qb = in_head / chunks, row0 = qb * bq + 32 * (in_head - qb * chunks);
  const int q_end = min(n_q, (qb + 1) * bq);
  if (row0 >= q_end) return;
  const int lane = threadIdx.x & 63, kz = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, h = lane >> 5;
  const uint64_t kbase = reinterpret_cast<uint64_t>(K + (size_t)bh * kv_stride * D);  // heads are kv_stride tokens apart
  const uint64_t vbase = reinterpret_cast<uint64_t>(V + (size_t)bh * kv_stride * D);
  const int32_t* row_idx = idx ? idx + ((size_t)bh * t_m + qb) * k : nullptr;
  const int nsel = idx ? k : t_n;
  const int subs = bkv >> 5;
  const int ntiles = nsel * subs;
  const int row = row0 + l32;            // rows past the block's end: clamped addresses, never written

  // the scaled queries sit in LDS, in the place of the first partial result (in registers they would leave no room for a
  // tile on its way); a piece is read one step ahead of its four products
  for (int e = threadIdx.x; e < 32 * (D / 4); e += 256) {
    const int rr = e / (D / 4), c4 = e - rr * (D / 4);
    *reinterpret_cast<f32x4*>(&part[0][rr][4 * c4]) =
        *reinterpret_cast<const f32x4*>(Q + ((size_t)bh * n_q + min(row0 + rr, n_q - 1)) * D + 4 * c4) * scale_log2e;
  }
  __syncthreads();
  const float* sq = &part[0][l32][4 * h];
  f32x4 qf = *reinterpret_cast<const f32x4*>(sq);
  auto score_step = [&](const f32x4& kpiece, int c, f32x16& acc) {   // qf holds piece c, and piece c + 1 (mod C) afterwards
    const f32x4 qn = *reinterpret_cast<const f32x4*>(sq + 8 * ((c + 1) % C));
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = mfma_f32_wide(kpiece[e], qf[e], acc);
    qf = qn;
  };
  f32x16 o[E];
#pragma unroll
  for (int e = 0; e < E; ++e)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[e][r] = 0.0f;
  float m = -INFINITY, l = 0.0f;

  // tile t of the list: first key and number of real keys (0: past the list or an index out of range)
  auto tile_at = [&](int t, int& first, int& cnt) {
    const int s = t / subs, sub = t - s * subs;
    const int jb = row_idx ? row_idx[min(s, nsel - 1)] : s;
    const int st = jb * bkv + 32 * sub;
    const bool ok = s < nsel && (unsigned)jb < (unsigned)t_n;
    const int n = ok ? min(32, n_kv - st) : 0;
    cnt = n > 0 ? n : 0;
    first = n > 0 ? st : 0;
  };
  auto desc = [&](uint64_t base, int first, int cnt) {
    const uint64_t b = base + (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane(first) * ROWB;
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(b), 0, __builtin_amdgcn_readfirstlane(cnt) * ROWB, 0x00020000);
  };
  int k_off = l32 * ROWB + 16 * h;
  int v_off[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) v_off[u] = (8 * u + 4 * h) * ROWB + 4 * E * l32;
  f32x4 kb[C];
  vpiece vb[16];
  auto load_k = [&](__amdgpu_buffer_rsrc_t d, int c) {
    kb[c] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(d, k_off + 32 * c, 0, 0));
  };
  auto load_v = [&](__amdgpu_buffer_rsrc_t d, int r) {
    const int off = v_off[r >> 2] + (r & 3) * ROWB;
    if constexpr (E == 4) vb[r] = __builtin_bit_cast(vpiece, __builtin_amdgcn_raw_buffer_load_b128(d, off, 0, 0));
    else vb[r] = __builtin_bit_cast(vpiece, __builtin_amdgcn_raw_buffer_load_b64(d, off, 0, 0));
  };

  f32x16 sc;   // scores of the wavefront's next tile
  // missing keys to -inf, the maximum into the reference m; what was accumulated under a smaller reference is scaled
  // (rarely: only once the maximum has grown by more than 2^8; any reference is exact in floating point)
  auto maxima = [&](int cnt) {
    if (cnt < 32) {
      const int mine = cnt - 4 * h;   // (one register; sixteen key numbers would be kept over the loop)
#pragma unroll
      for (int r = 0; r < 16; ++r) sc[r] = 8 * (r >> 2) + (r & 3) < mine ? sc[r] : -INFINITY;
    }
    float mx = sc[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, sc[r]);
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
    mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
    if (__any(mx > m + 8.0f)) {
      const float m_new = fmaxf(m, mx);
      const float alpha = exp2f(m - (m_new == -INFINITY ? 0.0f : m_new));
      m = m_new;
      l *= alpha;
#pragma unroll
      for (int e = 0; e < E; ++e)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[e][r] *= alpha;
    }
  };

  int first_v, cnt_v, first_k, cnt_k;
  tile_at(kz, first_v, cnt_v);
  tile_at(kz + KS, first_k, cnt_k);
  {
    const __amdgpu_buffer_rsrc_t dk = desc(kbase, first_v, cnt_v), dn = desc(kbase, first_k, cnt_k);
#pragma unroll
    for (int c = 0; c < C; ++c) load_k(dk, c);
#pragma unroll
    for (int r = 0; r < 16; ++r) sc[r] = 0.0f;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      score_step(kb[c], c, sc);
      load_k(dn, c);
      __builtin_amdgcn_sched_barrier(0);
    }
    maxima(cnt_v);
  }
  for (int t = kz; t < ntiles; t += KS) {
    const __amdgpu_buffer_rsrc_t dv = desc(vbase, first_v, cnt_v);
    int first_n, cnt_n;
    tile_at(t + 2 * KS, first_n, cnt_n);
    const __amdgpu_buffer_rsrc_t dk = desc(kbase, first_n, cnt_n);
    // (opaque here, or the sums of offsets leave the loop as sixteen registers instead of becoming immediates)
    asm volatile("" : "+v"(k_off), "+v"(v_off[0]), "+v"(v_off[1]), "+v"(v_off[2]), "+v"(v_off[3]));
    const float m_use = m == -INFINITY ? 0.0f : m;   // nothing seen yet: keep the exponents finite
    f32x16 p = sc;
#pragma unroll
    for (int r = 0; r < 16; ++r) sc[r] = 0.0f;
#pragma unroll
    for (int c = 0; c < C; ++c) {   // scores of tile t + KS; weights of tile t; its values requested
      score_step(kb[c], c, sc);
#pragma unroll
      for (int r = c * 16 / C; r < (c + 1) * 16 / C; ++r) {
        p[r] = __builtin_amdgcn_exp2f(p[r] - m_use);
        l += p[r];                  // this lane's keys only; summed at the end
        load_v(dv, r);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {  // tile t accumulated; the keys of tile t + 2 KS requested
#pragma unroll
      for (int e = 0; e < E; ++e) o[e] = mfma_f32_wide(vb[r][e], p[r], o[e]);
      if ((r + 1) * C / 16 > r * C / 16) load_k(dk, r * C / 16);
      __builtin_amdgcn_sched_barrier(0);
    }
    maxima(cnt_k);
    first_v = first_k;
    cnt_v = cnt_k;
    first_k = first_n;
    cnt_k = cnt_n;
  }

  // ---- weights of the KS parts of a row: w = 2^(m_part - m) / l
  auto both_halves = [](float x) {
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
  };
  l = both_halves(l);
  if (h == 0) {
    stat[l32][kz][0] = m;
    stat[l32][kz][1] = l;
  }
  __syncthreads();
  float m_tot = -INFINITY, l_tot = 0.0f;
#pragma unroll
  for (int u = 0; u < KS; ++u) m_tot = fmaxf(m_tot, stat[l32][u][0]);
  const float m_use = m_tot == -INFINITY ? 0.0f : m_tot;
#pragma unroll
  for (int u = 0; u < KS; ++u) l_tot = fmaf(stat[l32][u][1], exp2f(stat[l32][u][0] - m_use), l_tot);
  float w = l_tot > 0.0f ? exp2f(m - m_use) / l_tot : 0.0f;   // a row without a single real key: O_local = 0

  if (hist.lse2) {
    // ---- statistics for the backward pass: log2 of the sum of 2^(scaled logit), and D = dO . O_local from the unrounded
    // output, the four parts of which are summed as scalars
    const float* gp = static_cast<const float*>(hist.d_out) + ((size_t)bh * n_q + min(row, n_q - 1)) * D;
    float acc = 0.0f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const vpiece x = *reinterpret_cast<const vpiece*>(gp + E * (8 * (r >> 2) + 4 * h + (r & 3)));
#pragma unroll
      for (int e = 0; e < E; ++e) acc = fmaf(o[e][r] * w, x[e], acc);
    }
    acc = both_halves(acc);
    if (h == 0) part[0][l32][kz] = acc;
    __syncthreads();
    if (threadIdx.x < 32 && row < q_end) {
      const size_t at = (size_t)bh * n_q + row;
      hist.lse2[at] = l_tot > 0.0f ? m_tot + log2f(l_tot) : INFINITY;  // no real key: P = 0
      hist.dvec[at] = (part[0][l32][0] + part[0][l32][1]) + (part[0][l32][2] + part[0][l32][3]);
    }
    return;
  }

  float inv_den = 1.0f;
  if (hist.L) {
    // ---- O += R(phi(q)) L / (z_scale phi(q).z + eps) (Eq. 3, 6), as in attn_wide_kernel: O_local is scaled by the
    // denominator, the products add the numerator; wavefront kz takes the key features [kz D / 4, (kz + 1) D / 4)
    const float* L = hist.L + (size_t)bh * D * D;
    const float* z = hist.z + (size_t)bh * D + 4 * h;
    const float* qp = static_cast<const float*>(hist.q_hist) + ((size_t)bh * n_q + min(row, n_q - 1)) * D + 4 * h;
    const size_t trow = (size_t)min(row, n_q - 1) * (D / 2) + 2 * h;
    f32x4 ph[C / KS];
    float acc = 0.0f;
    auto features = [&](auto relu) {   // (one uniform choice of the feature map: a branch for every feature kept the loads apart)
#pragma unroll
      for (int c = 0; c < C; ++c) {
        f32x4 x = *reinterpret_cast<const f32x4*>(qp + 8 * c);
        const f32x4 zz = *reinterpret_cast<const f32x4*>(z + 8 * c);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          x[e] = phi_apply(x[e], relu.value ? HF_PHI_RELU : HF_PHI_ELU1);
          acc = fmaf(x[e], zz[e], acc);
        }
        if (c / (C / KS) == kz) ph[c % (C / KS)] = x;   // uniform
      }
    };
    if (hist.phi_kind == HF_PHI_RELU) features(std::true_type{}); else features(std::false_type{});
    if (hist.cosq) {
#pragma unroll
      for (int i = 0; i < C / KS; ++i) {
        const size_t at = trow + 4 * (kz * (C / KS) + i);
        const f32x2 cs = *reinterpret_cast<const f32x2*>(hist.cosq + at), sn = *reinterpret_cast<const f32x2*>(hist.sinq + at);
        ph[i] = rotate4(ph[i], cs[0], sn[0], cs[1], sn[1]);
      }
    }
    const float den = hist.z_scale * both_halves(acc) + hist.eps;
    w *= den;
    inv_den = 1.0f / den;
#pragma unroll
    for (int e = 0; e < E; ++e)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[e][r] *= w;
#pragma unroll
    for (int c = 0; c < C / KS; ++c) {
      const float* Lp = L + (size_t)(8 * (kz * (C / KS) + c) + 4 * h) * D + E * l32;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const vpiece a = *reinterpret_cast<const vpiece*>(Lp + (size_t)r * D);
#pragma unroll
        for (int e = 0; e < E; ++e) o[e] = mfma_f32_wide(a[e], ph[c][r], o[e]);
      }
    }
    w = 1.0f;
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    vpiece x;
#pragma unroll
    for (int e = 0; e < E; ++e) x[e] = o[e][r] * w * inv_den;
    *reinterpret_cast<vpiece*>(&part[kz][l32][E * (8 * (r >> 2) + 4 * h + (r & 3))]) = x;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < 32 * (D / 4); e += 256) {   // the four parts added, whole rows stored
    const int rr = e / (D / 4), c4 = e - rr * (D / 4);
    if (row0 + rr >= q_end) continue;
    f32x4 v = *reinterpret_cast<const f32x4*>(&part[0][rr][4 * c4]);
#pragma unroll
    for (int u = 1; u < KS; ++u) v += *reinterpret_cast<const f32x4*>(&part[u][rr][4 * c4]);
    *reinterpret_cast<f32x4*>(O + ((size_t)bh * n_q + row0 + rr) * D + 4 * c4) = v;
  }
}

template <int D>
int launch_wide32(const hf_config& c, const void* Q, int n_q, const void* K, const void* V, int n_kv, const int32_t* idx,
                  int k, void* O, const WideHist& hist, hipStream_t s) {
  const int t_m = (n_q + c.block_q - 1) / c.block_q, t_n = (n_kv + c.block_kv - 1) / c.block_kv;
  const long long total = (long long)c.batch * c.heads * t_m * (c.block_q / 32);
  if (total > (1ll << 30)) { set_error("too many query blocks"); return HF_ERR_SHAPE; }
  const int per_xcd = (int)((total + 7) / 8);
  const float scale = c.softmax_scale > 0.0f ? c.softmax_scale : 1.0f / sqrtf((float)c.head_dim);
  hipLaunchKernelGGL((attn_wide32_kernel<D>), dim3(8 * per_xcd), dim3(256), 0, s, static_cast<const float*>(Q),
                     static_cast<const float*>(K), static_cast<const float*>(V), idx, k, n_q, n_kv, kv_stride_of(c, n_kv),
                     c.block_q, c.block_kv, t_m, t_n, per_xcd, (int)total, scale * 1.4426950408889634f, hist,
                     static_cast<float*>(O));
  return check_launch("hf_hybrid_attn_fwd(attention)");
}

// Rows per workgroup: the most of 128, 64, 32, 16 that leaves at most an eighth of them without a query row and still gives
// two workgroups per compute unit; with fewer rows more wavefronts share them and a row's list is split further.
template <typename T, int D>
int launch_wide_rows(const hf_config& c, const void* Q, int n_q, const void* K, const void* V, int n_kv,
                     const int32_t* idx, int k, void* O, const WideHist& hist, hipStream_t s) {
  int rows = 128;
  while (rows > 16) {
    const int chunks = (c.block_q + rows - 1) / rows;
    const bool waste = chunks * rows * 8 > c.block_q * 9;       // more than an eighth of the rows do not exist
    const bool idle = row_groups(c, n_q, rows) < 512;           // fewer workgroups than two per compute unit
    if (!waste && !idle) break;
    rows >>= 1;
  }
  if (rows == 128) return launch_wide<T, D, 2, 1>(c, Q, n_q, K, V, n_kv, idx, k, O, hist, s);
  if (rows == 64) return launch_wide<T, D, 2, 2>(c, Q, n_q, K, V, n_kv, idx, k, O, hist, s);
  if (rows == 32) return launch_wide<T, D, 2, 4>(c, Q, n_q, K, V, n_kv, idx, k, O, hist, s);
  return launch_wide<T, D, 1, 4>(c, Q, n_q, K, V, n_kv, idx, k, O, hist, s);
}

}  // namespace

bool attn_d64_supported(const hf_config& c, int n_kv);   // hf_attn_d64.hip
int launch_attn_d64(const hf_config& c, const void* Q, int n_q, const void* K, const void* V, int n_kv, const int32_t* idx,
                    int k, void* O, const WideHist& hist, hipStream_t s);
bool attn_split_supported(const hf_config& c, int n_q, int n_kv);   // hf_attn_f32.hip
int launch_attn_split(const hf_config& c, const void* Q, int n_q, const void* K, const void* V, int n_kv, const int32_t* idx,
                      int k, void* O, const WideHist& hist, hipStream_t s);

static int launch_attn_wide(const hf_config& c, const void* Q, int n_q, const void* K, const void* V, int n_kv,
                            const int32_t* idx, int k, void* O, const WideHist& hist, hipStream_t s) {
  const long long keys = idx ? (long long)k * c.block_kv : n_kv;   // of a query row
  // bf16 at head_dim 64: the history term is a chain of loads and fp32 products behind the list, half as long with sixteen rows a
  // workgroup; behind a short list, in launches of few rows, that is what counts.  (Row statistics for the backward pass come from
  // the kernels of this file.)  Those against these, us, 2 to 64 blocks of 64 rows: with the term 64 keys 7.6..7.9 / 6.4..6.8, 128
  // 8.2..8.5 / 7.3..7.7, 256 9.5..9.8 / 9.2..9.8, 384 10.6..11.0 / 11.2..11.9; without 64 5.3..5.5 / 5.4..5.7, 256 7.1..7.3 / 8.1..8.6.
  const bool short_chain = hist.L && row_groups(c, n_q, 64) <= 64 && keys <= 256;
  if (attn_d64_supported(c, n_kv) && !hist.lse2 && !short_chain) return launch_attn_d64(c, Q, n_q, K, V, n_kv, idx, k, O, hist, s);
  if (attn_split_supported(c, n_q, n_kv)) return launch_attn_split(c, Q, n_q, K, V, n_kv, idx, k, O, hist, s);
  // fp32: 32 rows a workgroup or sixteen, in rounds of 256 compute units.  Up to 128 workgroups of 32 rows those of sixteen are one
  // round, up to 384 three (a second workgroup of 32 rows on a compute unit takes as long as two of sixteen more); between, they are
  // two for one, and pay where a list is short, whose chain they halve.  Sixteen / 32 rows, us, head_dim 128, history term off:
  // workgroups of 32 rows   14           120          132, 144     240          260          384          480
  //   64 keys               6.9 / 11.4   7.4 / 12.0   10.3 / 12.0  10.9 / 12.5  13.4 / 18.6  14.4 / 19.4  21.0 / 19.8
  //   192 keys              9.7 / 16.1   10.5 / 16.8  16.5 / 17.0  17.5 / 17.9  22.7 / 28.0  24.1 / 29.1  31.4 / 30.8
  //   384 keys              14.3 / 20.4  15.5 / 21.6  24.4 / 21.9  25.9 / 23.1  35.1 / 39.2  37.0 / 40.5  46.9 / 42.1
  //   1536 keys             42 / 55      50 / 61      70 / 61      74 / 66      101 / 111    107 / 115    142 / 123
  // (with the term and at head_dim 64 alike: 384 keys 14.1 / 13.2 at 144, 20.0 / 21.5 at 260, 21.2 / 22.2 at 384, 26.4 / 23.0 at 480)
  const long long wgs32 = row_groups(c, n_q, 32);
  const bool rows32 = wgs32 > 384 || (wgs32 > 128 && wgs32 <= 256 && keys > 192);
  if (c.dtype == HF_F32 && c.block_q % 32 == 0 && c.block_kv % 32 == 0 && rows32)
    return c.head_dim == 128 ? launch_wide32<128>(c, Q, n_q, K, V, n_kv, idx, k, O, hist, s)
                             : launch_wide32<64>(c, Q, n_q, K, V, n_kv, idx, k, O, hist, s);
  if (c.dtype == HF_F32)
    return c.head_dim == 128 ? launch_wide_rows<float, 128>(c, Q, n_q, K, V, n_kv, idx, k, O, hist, s)
                             : launch_wide_rows<float, 64>(c, Q, n_q, K, V, n_kv, idx, k, O, hist, s);
  return c.head_dim == 128 ? launch_wide_rows<bf16_t, 128>(c, Q, n_q, K, V, n_kv, idx, k, O, hist, s)
                           : launch_wide_rows<bf16_t, 64>(c, Q, n_q, K, V, n_kv, idx, k, O, hist, s);
}

int launch_attn_wide_stats(const hf_config& c, const void* Q, int n_q, const void* K, const void* V, int n_kv,
                           const int32_t* idx, int k, const void* dO, float* lse2, float* dvec, hipStream_t s) {
  WideHist h = {};
  h.lse2 = lse2;
  h.d_out = dO;
  h.dvec = dvec;
  return launch_attn_wide(c, Q, n_q, K, V, n_kv, idx, k, nullptr, h, s);
}

int launch_attn_mfma(const hf_config& c, const void* Q, int n_q, const void* K, const void* V, int n_kv,
                     const int32_t* idx, int k, void* O_local, hipStream_t s);  // hf_attn_mfma.hip
bool attn_mfma_supported(const hf_config& c);
int launch_attn_w64(const hf_config& c, const void* Q, int n_q, const void* K, const void* V, int n_kv,
                    const int32_t* idx, int k, void* O_local, hipStream_t s);  // hf_attn_w64.hip
bool attn_w64_supported(const hf_config& c);

// shapes whose attention kernel is the one of this file, which adds the history term itself
bool attn_wide_taken(const hf_config& c) { return !attn_mfma_supported(c) && !attn_w64_supported(c); }

// Steps of small fp32 streams as one launch: as many workgroups of sixteen rows as compute units at most.  Against selection and
// attention as launches of their own it gains by eight wavefronts on a list instead of four, and pays for a query block's mean by one
// wavefront of every workgroup, for the selection in front of the loop and for eight parts that meet.  A later step of one head,
// separate launches / this one, us, by tiles of 16 keys in a list: head_dim 128, blocks of 16: 2 tiles 12.1 / 12.7, 10 17.1 / 17.6, 20
// 21.6 / 21.8, 29 27.8 / 26.9, 64 38.7 / 33.6, 128 66.1 / 54.6; of 64: 4 12.9 / 13.5, 20 20.7 / 20.4, 40 29.3 / 26.3; head_dim 64,
// blocks of 16: 1 8.7 / 8.2, 16 11.9 / 11.1; where a chunk is too long to be pooled here on its later steps either, 24 19.2 / 20.1 (query
// blocks of 48) and 20.9 / 22.1 (of 512), 25 to 32 0.92 of the time.  (What is slower yet: the first step of a window that is pooled in
// front, with lists of a few tiles, 10.8 / 11.5 at the most; the later ones of its chunk gain.)
// Where the chunk's last step absorbs beside its attention, that step saves more than the others lose (head_dim 128, 8 heads, 16
// tokens: 15.7 / 13.0 the last, 12.8 / 12.9 the others; chunks of four steps 0.96 of the time in the mean of 83 sizes with lists that are
// too short otherwise, 1.03 at most).  Sums are in another order: the rule looks at what all steps of a chunk have in common, so that
// they run the same kernel, absorb or not.
bool attn_wide_step_supported(const hf_config& c, int n_q, int n_kv) {
  return c.dtype == HF_F32 && attn_wide_taken(c) && (n_kv + c.block_kv - 1) / c.block_kv <= kStepBlocks &&
         !attn_split_supported(c, n_q, n_kv) &&
         (long long)c.batch * c.heads * ((n_q + c.block_q - 1) / c.block_q) * ((c.block_q + 15) / 16) <= 256;
}
bool attn_wide_step_pays(const hf_config& c, int n_q, int k, bool absorbs) {
  const int tiles = k * ((c.block_kv + kTile - 1) / kTile);
  if (c.head_dim == 128) return absorbs || tiles >= 25 + c.block_q / 12;
  return absorbs || tiles > 24 || (n_q + c.block_kv - 1) / c.block_kv < kStepOwn;   // (a chunk touches a block more)
}
// Whether that launch pools the blocks [kv_first, kv_end) itself, every workgroup all of them, against a launch in front that pools each
// block once: by the bytes that a compute unit reads, beyond those that seven wavefronts get through while the eighth forms the query
// block's mean.  In the launch / in front of it, us: head_dim 128, 1 block of 64 (32 KB) 13.5 / 15.7, 8 (256 KB) 24.6 / 25.5; 12 of 128
// (768 KB) 29.9 / 27.6; 16 of 256 (2 MB) 38.9 / 30.9; 2 of 1024 (1 MB) 43.7 / 55.1, 8 (4 MB) 74.0 / 59.1; head_dim 64, 2 of 256 (128 KB)
// 12.2 / 15.2, 16 of 128 (512 KB) 15.6 / 14.5, 8 of 1024 (2 MB) 37.2 / 32.8.  Over 2324 sizes 0.06 % behind the better of the two.
bool attn_wide_step_pools(const hf_config& c, int kv_first, int kv_end) {
  const long long row = c.head_dim * (int)sizeof(float), bytes = (long long)(kv_end - kv_first) * c.block_kv * row;
  return kv_end - kv_first <= kStepOwn && bytes <= 256 * 1024 + 5 * c.block_q * row;
}
// Whether its workgroups absorb a chunk of n_ev tokens: of few enough heads for about one round of the chip, as far as LDS goes (a
// launch of its own has room for twice as many of them at head_dim 128).  The last step of a chunk, absorb behind it / in it, us,
// head_dim 128, 16 tokens: 8 heads 15.7 / 13.0, 48 17.8 / 18.1, 64 18.4 / 19.7, 128 24.5 / 27.7, 256 36.9 / 46.4; one token: 48 17.2 /
// 16.0, 64 17.5 / 18.0; head_dim 64, 256 heads 15.2 / 15.0.
bool attn_wide_step_absorbs(const hf_config& c, int n_ev) {
  const long long workgroups = (long long)c.batch * c.heads * (c.head_dim / 32) * (c.head_dim / 32);
  return n_ev <= kAbsorbOneSlice && workgroups <= (c.head_dim == 128 ? 768 : 1024);
}

int launch_attn_wide_step(const hf_config& c, const void* Q, const void* Q_hist, int n_q, const void* K, const void* V, int n_kv, int k,
                          const float* state, const float* cosq, const float* sinq, float* kbar_t, int32_t* idx_out, int kv_first,
                          int kv_end, void* O, const void* K_ev, const void* V_ev, int n_ev, int ev_stride, const float* cos_ev,
                          const float* sin_ev, float* state_out, hipStream_t s) {
  const size_t d = c.head_dim;
  WideHist h = {};
  h.phi_kind = c.phi;
  if (state) {
    h.L = state;
    h.z = state + (size_t)c.batch * c.heads * d * d;
    h.cosq = cosq;
    h.sinq = sinq;
    h.q_hist = Q_hist;
    h.eps = c.eps;
    h.z_scale = c.z_scale;
  }
  WideStep st = {};
  st.kbar_t = kbar_t;
  st.idx_out = idx_out;
  st.kv_first = kv_first;
  st.kv_end = kv_end;
  st.K_ev = K_ev;
  st.V_ev = V_ev;
  st.n_ev = n_ev;
  st.ev_stride = ev_stride;
  st.cos_ev = cos_ev;
  st.sin_ev = sin_ev;
  st.state_in = state;
  st.state_out = state_out;
  return c.head_dim == 128 ? launch_wide_step_d<128>(c, Q, n_q, K, V, n_kv, k, O, h, st, s)
                           : launch_wide_step_d<64>(c, Q, n_q, K, V, n_kv, k, O, h, st, s);
}

int launch_attn_wide_hist(const hf_config& c, const void* Q, const void* Q_hist, int n_q, const void* K, const void* V,
                          int n_kv, const int32_t* idx, int k, const float* state, const float* cosq, const float* sinq,
                          void* O, hipStream_t s) {
  WideHist h = {};
  h.L = state;
  h.z = state + (size_t)c.batch * c.heads * c.head_dim * c.head_dim;
  h.cosq = cosq;
  h.sinq = sinq;
  h.q_hist = Q_hist;
  h.eps = c.eps;
  h.z_scale = c.z_scale;
  h.phi_kind = c.phi;
  return launch_attn_wide(c, Q, n_q, K, V, n_kv, idx, k, O, h, s);
}

int launch_attn(const hf_config& c, const void* Q, int n_q, const void* K, const void* V, int n_kv,
                const int32_t* idx, int k, void* O_local, hipStream_t s) {
  // bf16, head_dim 128: block_q 64 / 128 take the workgroup-per-query-block MFMA kernel, other
  // multiples of 64 the wavefront-per-64-rows MFMA kernel; everything else the fp32-arithmetic one
  if (attn_mfma_supported(c)) return launch_attn_mfma(c, Q, n_q, K, V, n_kv, idx, k, O_local, s);
  if (attn_w64_supported(c)) return launch_attn_w64(c, Q, n_q, K, V, n_kv, idx, k, O_local, s);
  return launch_attn_wide(c, Q, n_q, K, V, n_kv, idx, k, O_local, WideHist{}, s);
}

}  // namespace hf
