// Gradients of the hybrid attention for the training algorithm of the supplement (the one step per
// chunk that runs with gradients enabled): dQ, dK, dV of the block-sparse softmax attention (Eq. 5)
// for a fixed Top-K mask, and the gradient of the history readout (Eq. 3) with respect to its
// queries for a constant state.  This file: the kernels every shape and type can take (fp32
// arithmetic on the fp32 matrix instruction, hf_f32_mfma.h) and the small helpers shared with the bf16 path.
//
// With P recomputed from the saved row statistic lse2 = log2 sum_j 2^(c s_ij) (c = scale log2 e):
//     D_i  = dO_i . O_local_i = sum_j P_ij dP_ij   (with stored scores the sum; else the product, from the recomputed forward
//                                                    pass, before O_local is rounded)
//     dV_j = sum_i P_ij dO_i               dP_ij = dO_i . v_j
//     dS_ij = P_ij (dP_ij - D_i)
//     dQ_i = scale sum_j dS_ij k_j         dK_j = scale sum_i dS_ij q_i
// dQ walks the index list of its query block; dK, dV walk the inverse list (the query blocks that
// selected a KV block), so both accumulate in registers and nothing is added atomically.
#include <float.h>
#include <math.h>

#include "hf_f32_mfma.h"

namespace hf {
namespace {

// ---- inverse of the index lists: for every KV block the query blocks whose row holds it, ascending ----
// One wavefront per (head, KV block): lane = query block, 64 at a time; a ballot and a prefix count compact
// the hits in order.
__global__ __launch_bounds__(256) void invert_index_kernel(const int32_t* __restrict__ idx, int k, int t_m, int t_n,
                                                           int32_t* __restrict__ inv_cnt,
                                                           int32_t* __restrict__ inv_list,
                                                           int32_t* __restrict__ inv_slot) {
  const int lane = threadIdx.x & 63;
  const int j = blockIdx.x * 4 + (threadIdx.x >> 6), bh = blockIdx.y;
  if (j >= t_n) return;
  const int32_t* rows = idx + (size_t)bh * t_m * k;
  int32_t* out = inv_list + ((size_t)bh * t_n + j) * t_m;
  int32_t* slots = inv_slot ? inv_slot + ((size_t)bh * t_n + j) * t_m : nullptr;
  int cnt = 0;
  for (int i0 = 0; i0 < t_m; i0 += kWave) {
    const int i = i0 + lane;
    int at = -1;
    if (i < t_m)
      for (int s = 0; s < k; ++s) at = rows[(size_t)i * k + s] == j ? s : at;   // by contract a row lists a block at most once
    const unsigned long long mask = __ballot(at >= 0);
    if (at >= 0) {
      const int place = cnt + __popcll(mask & ((1ull << lane) - 1ull));
      out[place] = i;
      if (slots) slots[place] = at;
    }
    cnt += __popcll(mask);
  }
  if (lane == 0) inv_cnt[(size_t)bh * t_n + j] = cnt;
}

// ---- what the gradient kernels need prepared, in one launch (each part alone is shorter than a launch costs): workgroups
// take a part by their number.
//
//   order   one per XCD's share of the dK/dV items: launch order, see below
//   invert  one per head: the inverse lists
//   planes  two 32 x 32 tiles of a head's state each: fp32 -> the bf16 planes L^T and L of the history branch's gradient
//   dots    32 rows each: D = dO . O_local from a saved O_local
//
// 832x480 (12 heads, 4680 x 9360, blocks of 64, k = 37): 11.1 us, where launches of their own took 7.4 + 6.2 + 5.0 + 6.7 us
// and three gaps; the whole training step 395 -> 382 us, one of 35 heads x 282 tokens 72.4 -> 65.7 us.
constexpr int kPrepThreads = 512;
struct PrepArgs {
  const int32_t* idx;            // [BH][t_m][k]
  int k, t_m, t_n;
  int order_wgs, invert_wgs, plane_wgs;
  int32_t *inv_cnt, *inv_list;   // [BH][t_n], [BH][t_n][t_m]
  int32_t* inv_slot;             // [BH][t_n][t_m] or NULL: the block's place in the row of each query block on its list
  int slabs, items_per_xcd, total_items;
  int32_t* order;                // [8 items_per_xcd][kOrderRec]
  const float* state;
  bf16_t* planes;
  const bf16_t *A, *B;
  long long rows;
  float* dots;
};

// every entry of the index rows of the heads that KV blocks [b0, b0 + n) (numbered over all heads) belong to, every thread
// its share: f(block - b0, query block, place in the row) for the entries that lie in the range
template <typename F>
__device__ __forceinline__ void each_entry(const PrepArgs& p, int b0, int n, F f) {
  const int tid = threadIdx.x;
  const int row_words = p.t_m * p.k;   // entries of a head
  const int h0 = b0 / p.t_n, entries = ((b0 + n - 1) / p.t_n - h0 + 1) * row_words;
  const int32_t* src = p.idx + (size_t)h0 * row_words;
  const uint32_t per_k = 0xffffffffu / (uint32_t)p.k + 1u;   // e / k = e per_k / 2^32, as e k < t_m k^2 < 2^32
  constexpr int U = 8;                 // entries in flight per thread: the pass is round trips to memory
  for (int e0 = tid; e0 < entries; e0 += U * kPrepThreads) {
    int entry[U];
#pragma unroll
    for (int u = 0; u < U; ++u) entry[u] = src[min(e0 + u * kPrepThreads, entries - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      int e = e0 + u * kPrepThreads, at = h0 * p.t_n - b0;
      if (e >= entries) break;
      while (e >= row_words) {         // (the blocks of a share belong to a few heads)
        e -= row_words;
        at += p.t_n;
      }
      const int j = entry[u], i = p.k == 1 ? e : (int)__umulhi((uint32_t)e, per_k);
      if ((unsigned)j < (unsigned)p.t_n && (unsigned)(at + j) < (unsigned)n) f(at + j, i, e - i * p.k);
    }
  }
}

// The inverse lists as bit masks in LDS: for KV blocks [b0, b0 + n) one bit per query block that selected it, 32 to a word.
// A block's list is then the positions of its bits, its length their number, and bit i stands at the number of bits below it.
__device__ __forceinline__ void selected_by(uint32_t* mask, const PrepArgs& p, int b0, int n, int words) {
  for (int e = threadIdx.x; e < n * words; e += kPrepThreads) mask[e] = 0;
  __syncthreads();
  each_entry(p, b0, n, [&](int block, int i, int) { atomicOr(&mask[block * words + (i >> 5)], 1u << (i & 31)); });
  __syncthreads();
}

// bucket[len] = number of items of a length, 0 .. longest -> where they start: exclusive sums from the longest down
__device__ __forceinline__ void starts_from_longest(int32_t* bucket, int longest) {
  const int tid = threadIdx.x;
  if (tid < kWave) {
    int before = 0;
    for (int top = longest; top >= 0; top -= kWave) {
      const int own = top - tid >= 0 ? bucket[top - tid] : 0;
      int sum = own;
#pragma unroll
      for (int o = 1; o < kWave; o <<= 1) {
        const int up = __shfl_up(sum, o, kWave);
        if (tid >= o) sum += up;
      }
      if (top - tid >= 0) bucket[top - tid] = before + sum - own;
      before += __shfl(sum, kWave - 1, kWave);
    }
  }
  __syncthreads();
}

// Launch order of the dK/dV workgroups.  A workgroup's time is proportional to the length of its KV block's list of query
// blocks, and the lists differ (top-k selection: a binomial spread around t_m k / t_n), while a GPU takes workgroups in index
// order as slots free up.  Longest first within every XCD's share of the items leaves the short ones to fill the end.  One
// record of kOrderRec words per place: the item that runs there, the length of its list and the list's first three entries,
// so that a workgroup has all it needs for its first tiles after ONE dependent load (it is alone on its two SIMDs: every
// round trip to memory before its first MFMA is idle time).  The masks are formed here once more, for the share's blocks:
// waiting for the workgroups that write the lists would take another launch.
__device__ __forceinline__ void order_share(int32_t* smem, const PrepArgs& p, int share, int words) {
  const int first = share * p.items_per_xcd;
  const int n = min(p.items_per_xcd, p.total_items - first);
  if (n <= 0) return;
  const int b0 = first / p.slabs, nb = (first + n - 1) / p.slabs - b0 + 1;   // KV blocks (of all heads) of the share
  int32_t* const key = smem;                                                  // [n] list length
  int32_t* const bucket = key + p.items_per_xcd;                              // [t_m + 1] items of a length; their places
  uint32_t* const mask = reinterpret_cast<uint32_t*>(bucket + p.t_m + 1);     // [nb][words]
  const int tid = threadIdx.x;
  for (int e = tid; e <= p.t_m; e += kPrepThreads) bucket[e] = 0;
  selected_by(mask, p, b0, nb, words);
  for (int j = tid; j < n; j += kPrepThreads) {
    const uint32_t* m = mask + ((first + j) / p.slabs - b0) * words;
    int len = 0;
    for (int w = 0; w < words; ++w) len += __popc(m[w]);
    key[j] = len;
    atomicAdd(&bucket[len], 1);
  }
  __syncthreads();
  starts_from_longest(bucket, p.t_m);
  for (int j = tid; j < n; j += kPrepThreads) {
    const uint32_t* m = mask + ((first + j) / p.slabs - b0) * words;
    int entry[3] = {0, 0, 0}, w = 0;
    uint32_t bits = m[0];
#pragma unroll
    for (int q = 0; q < 3; ++q)
      if (q < key[j]) {
        while (!bits) bits = m[++w];   // (key[j] bits are set: ends)
        entry[q] = 32 * w + __ffs(bits) - 1;
        bits &= bits - 1;
      }
    // (which of two equally long lists comes first does not matter: every item runs once, whatever its place)
    int4* rec = reinterpret_cast<int4*>(p.order + (size_t)(first + atomicAdd(&bucket[key[j]], 1)) * kOrderRec);
    rec[0] = int4{first + j, key[j], entry[0], entry[1]};
    rec[1] = int4{entry[2], 0, 0, 0};
  }
}

__global__ __launch_bounds__(kPrepThreads) void bwd_prep_kernel(PrepArgs p) {
  extern __shared__ int32_t prep_smem[];
  int wg = blockIdx.x;
  const int words = (p.t_m + 31) >> 5;
  if (wg < p.order_wgs) {
    order_share(prep_smem, p, wg, words);
    return;
  }
  wg -= p.order_wgs;
  if (wg < p.invert_wgs) {
    uint32_t* const mask = reinterpret_cast<uint32_t*>(prep_smem);
    selected_by(mask, p, wg * p.t_n, p.t_n, words);
    int32_t* const out = p.inv_list + (size_t)wg * p.t_n * p.t_m;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int j = wave; j < p.t_n; j += kPrepThreads / 64) {   // a wavefront per list, two words of its mask at a time
      const uint32_t* m = mask + j * words;
      int below = 0;
      for (int w = 0; w < words; w += 2) {
        const unsigned long long both = m[w] | (w + 1 < words ? (unsigned long long)m[w + 1] << 32 : 0ull);
        if (both >> lane & 1ull) out[(size_t)j * p.t_m + below + __popcll(both & ((1ull << lane) - 1ull))] = 32 * w + lane;
        below += __popcll(both);
      }
      if (lane == 0) p.inv_cnt[(size_t)wg * p.t_n + j] = below;
    }
    if (p.inv_slot) {
      int32_t* const slots = p.inv_slot + (size_t)wg * p.t_n * p.t_m;
      each_entry(p, wg * p.t_n, p.t_n, [&](int j, int i, int slot) {
        const uint32_t* m = mask + j * words;
        int below = __popc(m[i >> 5] & ((1u << (i & 31)) - 1u));
        for (int w = 0; w < i >> 5; ++w) below += __popc(m[w]);
        slots[(size_t)j * p.t_m + below] = slot;
      });
    }
    return;
  }
  wg -= p.invert_wgs;
  const int tid = threadIdx.x;
  if (wg < p.plane_wgs) {
    constexpr int D = 128;
    const int half = tid >> 8, t = tid & 255, tx = t & 31, ty = t >> 5;   // 32 x 8 threads per tile
    float* tile = reinterpret_cast<float*>(prep_smem) + half * 32 * 33;
    const int bh = wg >> 3, which = 2 * (wg & 7) + half, i0 = 32 * (which >> 2), j0 = 32 * (which & 3);
    const float* L = p.state + (size_t)bh * D * D;
    bf16_t* lt = p.planes + (size_t)bh * 2 * D * D;
    bf16_t* ln = lt + D * D;
    for (int r = ty; r < 32; r += 8) {
      const float v = L[(size_t)(i0 + r) * D + j0 + tx];
      tile[r * 33 + tx] = v;
      ln[(size_t)(i0 + r) * D + j0 + tx] = f32_to_bf16(v);
    }
    __syncthreads();
    for (int r = ty; r < 32; r += 8) lt[(size_t)(j0 + r) * D + i0 + tx] = f32_to_bf16(tile[tx * 33 + r]);
    return;
  }
  wg -= p.plane_wgs;
  // 16 lanes per row, 16 bytes per lane and tensor, fp32 arithmetic
  const long long row = (long long)wg * (kPrepThreads / 16) + (tid >> 4);
  const int part = tid & 15;
  float acc = 0.0f;
  if (row < p.rows) {
    const uint4 a = *reinterpret_cast<const uint4*>(p.A + row * 128 + part * 8);
    const uint4 b = *reinterpret_cast<const uint4*>(p.B + row * 128 + part * 8);
    const uint32_t aw[4] = {a.x, a.y, a.z, a.w}, bw[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      acc = fmaf(__uint_as_float(aw[i] << 16), __uint_as_float(bw[i] << 16), acc);
      acc = fmaf(__uint_as_float(aw[i] & 0xffff0000u), __uint_as_float(bw[i] & 0xffff0000u), acc);
    }
  }
#pragma unroll
  for (int off = 8; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 16);
  if (row < p.rows && part == 0) p.dots[row] = acc;
}

// The same order from finished lists, in a launch behind them, where a share's masks do not fit in LDS (long windows).  Lengths
// go to kLengths buckets, several to one where a list can be longer than that.  Gradients of 8 heads, 1024 query and 1150 KV
// blocks of 64, k = 64: 5.73 ms in index order, 4.00 with this launch.
constexpr int kLengths = 8192;
constexpr int kOrderThreads = 1024;
__global__ __launch_bounds__(kOrderThreads) void dkv_order_kernel(const int32_t* __restrict__ inv_cnt,
                                                                  const int32_t* __restrict__ inv_list, int t_m, int slabs,
                                                                  int items_per_xcd, int total_items, int shift,
                                                                  int32_t* __restrict__ order) {
  __shared__ int32_t bucket[kLengths];
  const int first = blockIdx.x * items_per_xcd, n = min(items_per_xcd, total_items - first), tid = threadIdx.x;
  if (n <= 0) return;
  for (int e = tid; e <= t_m >> shift; e += kOrderThreads) bucket[e] = 0;
  __syncthreads();
  for (int j = tid; j < n; j += kOrderThreads) atomicAdd(&bucket[inv_cnt[(first + j) / slabs] >> shift], 1);
  __syncthreads();
  starts_from_longest(bucket, t_m >> shift);
  for (int j = tid; j < n; j += kOrderThreads) {
    const int kvb = (first + j) / slabs, len = inv_cnt[kvb];
    const int32_t* list = inv_list + (size_t)kvb * t_m;
    int entry[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) entry[q] = q < len ? list[q] : 0;
    int4* rec = reinterpret_cast<int4*>(order + (size_t)(first + atomicAdd(&bucket[len >> shift], 1)) * kOrderRec);
    rec[0] = int4{first + j, len, entry[0], entry[1]};
    rec[1] = int4{entry[2], 0, 0, 0};
  }
}

// History branch (Eq. 3) in the dQ kernel's epilogue, as in the bf16 kernel: with f = phi(q), r = R f,
// den = z_scale f.z + eps, num = r L:   dnum = g / den, dden = -(g . num) / den^2,
// dq = (R^T (dnum L^T) + z_scale dden z) phi'(q)
struct WideBwdHist {
  const float* L;        // [BH][D][D], NULL: none
  const float* z;        // [BH][D]
  const float* cosq;     // [n_q][D/2] or NULL
  const float* sinq;
  const void* q_hist;    // [BH][n_q][D] queries of the history branch
  void* dq_hist;         // given: their gradient on its own; NULL: it joins dQ before the one rounding
  float eps, z_scale;
  int phi_kind;
};

constexpr int kParts = 4;   // wavefronts of a workgroup: they share its rows (keys) and split the list between them

constexpr int kStoredWaves = 8;   // of a workgroup that works from stored scores

// The parts of a [16 N][D] result (column-form accumulators, FW pieces of 64 features from 64 f0 on) meet in LDS, AT_ONCE of
// PARTS at a time: [AT_ONCE][16 N][D + 4].  on_top (uniform): the first's place holds something that is added to.
template <int D, int N, int PARTS, int AT_ONCE, int FW>
__device__ __forceinline__ void add_parts(float* smem, const f32x4 (&acc)[N][FW][4], float mul, bool on_top, int part, int f0, int l16,
                                          int g) {
  constexpr int OST = D + 4, TURNS = PARTS / AT_ONCE;
  float* const own = smem + ((part % AT_ONCE) * 16 * N + l16) * OST + 64 * f0 + 16 * g;
#pragma unroll
  for (int turn = TURNS - 1; turn >= 0; --turn) {
    if (part / AT_ONCE == turn)   // uniform
#pragma unroll
      for (int n = 0; n < N; ++n)
#pragma unroll
        for (int f = 0; f < FW; ++f)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            f32x4* const at = reinterpret_cast<f32x4*>(own + 16 * n * OST + 64 * f + 4 * r);
            const f32x4 v = f32x4{acc[n][f][0][r], acc[n][f][1][r], acc[n][f][2][r], acc[n][f][3][r]} * mul;
            *at = turn < TURNS - 1 || (on_top && part % AT_ONCE == 0) ? v + *at : v;
          }
    __syncthreads();
  }
}
// ... and whole rows are stored
template <typename T, int D, int N, int AT_ONCE, int WAVES>
__device__ __forceinline__ void store_parts(const float* smem, T* dst, int rows, int tid) {
  constexpr int OST = D + 4;
  for (int e = tid; e < 16 * N * (D / 4); e += 64 * WAVES) {
    const int rr = e / (D / 4), c4 = e - rr * (D / 4);
    if (rr >= rows) continue;
    f32x4 v = *reinterpret_cast<const f32x4*>(smem + (size_t)rr * OST + 4 * c4);
#pragma unroll
    for (int u = 1; u < AT_ONCE; ++u) v += *reinterpret_cast<const f32x4*>(smem + ((size_t)u * 16 * N + rr) * OST + 4 * c4);
    store4<T>(dst + (size_t)rr * D + 4 * c4, v);
  }
}

struct WideBwd {
  const void *Q, *K, *V, *dO;
  const int32_t* idx;                              // [BH][t_m][k] or NULL (dense: k = t_n)
  int k, n_q, n_kv, kv_stride, bq, bkv, t_m, t_n;
  int q_chunks, q_per_xcd, q_total;                // workgroups of the query side: chunks of a block, items of an XCD's share, items
  int k_chunks, k_per_xcd, k_total;                // of the key side
  const int32_t* order;                            // stored scores: KV blocks, longest list first (records of kOrderRec), or NULL
  float scale_log2e, scale;
  float *lse2, *Dv;                                // [BH][n_q]
  const int32_t *inv_cnt, *inv_list, *inv_slot;    // [BH][t_n], [BH][t_n][t_m]; dense: NULL
  float* scores;                                   // stored scores, see bwd_scores_kernel
  WideBwdHist hist;
  void *dQ, *dK, *dV;
};

// Stored scores: a panel per (query block, place of its list), a panel's tiles of 16 queries x 16 keys row by row, a tile's S
// [query][key] (times scale log2 e) and then its dP.
constexpr int kScoreTile = 2 * 16 * 16;
constexpr size_t kScoresRoom = (size_t)2 << 30;   // most that a workspace holds of them
__device__ __forceinline__ const float* score_tile(const WideBwd& a, int bh, int qb, int slot, int qi, int ki) {
  const int qt = (a.bq + 15) / 16, kt = (a.bkv + 15) / 16;
  return a.scores + ((((size_t)bh * a.t_m + qb) * a.k + slot) * (qt * kt) + qi * kt + ki) * kScoreTile;
}

// ---- S^T = K Q^T and dP^T = V dO^T, once for all three gradients: a workgroup per 16 NQ query rows, its eight wavefronts
// splitting the list; both go to memory as fp32 (score_tile), and lse2 and D = sum_j P_ij dP_ij leave with them, so that no
// forward pass is formed again: five products of the forward's size instead of nine (two of the statistics, three for dQ, four
// for dK and dV).  Statistics are a lane's own until the end: maximum, sum and weighted sum over the keys it holds.
// Bound by the fp32 matrix rate at the clock it holds (2.0 GHz): 12 heads of 128, 1170 x 2340, k = 10 of 37 blocks of 64: 58 us,
// the pipes 66 % busy while a compute unit has work (456 workgroups for 512 places); with the gradients behind it (95) instead of
// statistics (42), dQ (93) and dK, dV (122): 74 training steps 0.60 to 0.87 of the time, 0.69 in the mean.  Errors against 64 bits
// are no larger (dQ 6.1e-7 -> 6.0e-7, with four times the queries 2.8e-6 -> 1.4e-6).
constexpr int kScoreParts = 8;
template <typename T, int D, int NQ>
__global__ __launch_bounds__(64 * kScoreParts, 4) void bwd_scores_kernel(WideBwd a) {
  constexpr int ROWS = 16 * NQ, C = D / 16, OST = D + 4;
  extern __shared__ __attribute__((aligned(16))) float smem[];   // [ROWS][OST] Q, [ROWS][OST] dO
  __shared__ float stat[3][kScoreParts][ROWS];
  float* sQ = smem;
  float* sG = smem + ROWS * OST;
  const int wg = blockIdx.x, item = (wg & 7) * a.q_per_xcd + (wg >> 3);
  if ((wg >> 3) >= a.q_per_xcd || item >= a.q_total) return;
  const int n_q = a.n_q, n_kv = a.n_kv, bq = a.bq, bkv = a.bkv, t_n = a.t_n;
  const int bh = item / (a.t_m * a.q_chunks), in_head = item - bh * a.t_m * a.q_chunks;
  const int qb = in_head / a.q_chunks, row0 = qb * bq + (in_head - qb * a.q_chunks) * ROWS;
  const int q_end = min(n_q, (qb + 1) * bq);
  if (row0 >= q_end) return;
  const int lane = threadIdx.x & 63, kz = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  const T* __restrict__ Q = static_cast<const T*>(a.Q);
  const T* __restrict__ dO = static_cast<const T*>(a.dO);
  const T* __restrict__ Kh = static_cast<const T*>(a.K) + (size_t)bh * a.kv_stride * D;
  const T* __restrict__ Vh = static_cast<const T*>(a.V) + (size_t)bh * a.kv_stride * D;
  const int32_t* __restrict__ row_idx = a.idx ? a.idx + ((size_t)bh * a.t_m + qb) * a.k : nullptr;
  const int nsel = a.idx ? a.k : t_n, subs = (bkv + 15) / 16, ntiles = nsel * subs;
  const int qt = (bq + 15) / 16, qi0 = (row0 - qb * bq) / 16;
  for (int e = threadIdx.x; e < ROWS * (D / 4); e += 64 * kScoreParts) {
    const int rr = e / (D / 4), c4 = e - rr * (D / 4);
    const size_t off = ((size_t)bh * n_q + min(row0 + rr, n_q - 1)) * D + 4 * c4;
    *reinterpret_cast<f32x4*>(sQ + rr * OST + 4 * c4) = load4<T>(Q + off) * a.scale_log2e;
    *reinterpret_cast<f32x4*>(sG + rr * OST + 4 * c4) = load4<T>(dO + off);
  }
  __syncthreads();
  auto tile_at = [&](int t, int& first, int& cnt) {   // cnt 0: past the list, an index out of range, or no such keys
    const int s = t / subs, sub = t - s * subs;
    const int jb = row_idx ? row_idx[min(s, nsel - 1)] : s;
    const int st = jb * bkv + 16 * sub;
    const bool ok = s < nsel && (unsigned)jb < (unsigned)t_n;
    const int n = ok ? min(16, min(n_kv, (jb + 1) * bkv) - st) : 0;
    cnt = n > 0 ? n : 0;
    first = n > 0 ? st : 0;
  };
  constexpr int B = sizeof(T);
  int row_at = (l16 * D + 4 * g) * B;   // rows behind a tile's last real key read as zeros
  Piece<T> kr[C], vr[C];
  int first, cnt, first_n, cnt_n;
  tile_at(kz, first, cnt);
  {
    const __amdgpu_buffer_rsrc_t k_rows = tile_rows<T, D>(Kh, first, cnt), v_rows = tile_rows<T, D>(Vh, first, cnt);
#pragma unroll
    for (int c = 0; c < C; ++c) {
      kr[c].load(k_rows, row_at + 16 * c * B);
      vr[c].load(v_rows, row_at + 16 * c * B);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  float m[NQ], l[NQ], d[NQ];
#pragma unroll
  for (int n = 0; n < NQ; ++n) {
    m[n] = -FLT_MAX;
    l[n] = d[n] = 0.0f;
  }
  const float* bq0 = sQ + l16 * OST + 4 * g;
  const float* bg0 = sG + l16 * OST + 4 * g;
  for (int t = kz; t < ntiles; t += kScoreParts) {
    asm volatile("" : "+v"(row_at));   // (opaque here, or its sums leave the loop as registers instead of immediates)
    tile_at(t + kScoreParts, first_n, cnt_n);
    const __amdgpu_buffer_rsrc_t kn_rows = tile_rows<T, D>(Kh, first_n, cnt_n), vn_rows = tile_rows<T, D>(Vh, first_n, cnt_n);
    f32x4 s[NQ], p[NQ];
#pragma unroll
    for (int n = 0; n < NQ; ++n) s[n] = p[n] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const f32x4 ka = kr[c].get(), va = vr[c].get();
      f32x4 b[NQ], gg[NQ];
#pragma unroll
      for (int n = 0; n < NQ; ++n) {
        b[n] = *reinterpret_cast<const f32x4*>(bq0 + 16 * n * OST + 16 * c);
        gg[n] = *reinterpret_cast<const f32x4*>(bg0 + 16 * n * OST + 16 * c);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int n = 0; n < NQ; ++n) {
          s[n] = mfma_f32(ka[e], b[n][e], s[n]);
          p[n] = mfma_f32(va[e], gg[n][e], p[n]);
        }
      kr[c].load(kn_rows, row_at + 16 * c * B);
      vr[c].load(vn_rows, row_at + 16 * c * B);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (cnt > 0) {   // uniform
      const int slot = t / subs;
#pragma unroll
      for (int n = 0; n < NQ; ++n) {
        if (cnt < 16)   // keys that do not exist: probability zero
#pragma unroll
          for (int r = 0; r < 4; ++r) s[n][r] = 4 * g + r < cnt ? s[n][r] : -__builtin_inff();
        if (qi0 + n < qt) {
          float* tile = const_cast<float*>(score_tile(a, bh, qb, slot, qi0 + n, t - slot * subs)) + 16 * l16 + 4 * g;
          *reinterpret_cast<f32x4*>(tile) = s[n];
          *reinterpret_cast<f32x4*>(tile + kScoreTile / 2) = p[n];
        }
        const float top = fmaxf(fmaxf(fmaxf(s[n][0], s[n][1]), fmaxf(s[n][2], s[n][3])), m[n]);
        const float kept = __builtin_amdgcn_exp2f(m[n] - top);
        float sum = 0.0f, weighted = 0.0f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float w = __builtin_amdgcn_exp2f(s[n][r] - top);
          sum += w;
          weighted = fmaf(w, p[n][r], weighted);
        }
        l[n] = fmaf(l[n], kept, sum);
        d[n] = fmaf(d[n], kept, weighted);
        m[n] = top;
      }
    }
    cnt = cnt_n;
  }
#pragma unroll
  for (int n = 0; n < NQ; ++n) {
    const float top = column_max(m[n]), w = __builtin_amdgcn_exp2f(m[n] - top);
    const float sum = column_sum(l[n] * w), weighted = column_sum(d[n] * w);
    if (g == 0) {
      stat[0][kz][16 * n + l16] = top;
      stat[1][kz][16 * n + l16] = sum;
      stat[2][kz][16 * n + l16] = weighted;
    }
  }
  __syncthreads();
  const int rr = threadIdx.x;
  if (rr < ROWS && row0 + rr < q_end) {
    float top = stat[0][0][rr], sum = 0.0f, weighted = 0.0f;
#pragma unroll
    for (int u = 1; u < kScoreParts; ++u) top = fmaxf(top, stat[0][u][rr]);
#pragma unroll
    for (int u = 0; u < kScoreParts; ++u) {
      const float w = __builtin_amdgcn_exp2f(stat[0][u][rr] - top);
      sum = fmaf(stat[1][u][rr], w, sum);
      weighted = fmaf(stat[2][u][rr], w, weighted);
    }
    const size_t at = (size_t)bh * n_q + row0 + rr;
    // no key at all (an empty list), or a sum that is no number: probabilities are zero, so that the row adds nothing to the values'
    // gradients of its other keys, as where every kernel forms its own scores
    a.lse2[at] = sum > 0.0f ? top + __builtin_amdgcn_logf(sum) : __builtin_inff();
    a.Dv[at] = sum == 0.0f ? 0.0f : weighted / sum;
  }
}

// Gradient of the history branch with respect to its queries, for the workgroup's rows (dO in sG; sQ is written): to dq_hist
// where it is given, else sink(n, f, pr, r, v0, v1) has the values of row 16 n + l % 16, features 64 f + 16 (l / 16) + 4 r + 2 pr, + 1.
template <typename T, int D, int NQ, int WAVES, typename Sink>
__device__ __forceinline__ void history_gradient(const WideBwdHist& hist, int bh, int row0, int q_end, int n_q, int kz, int l16,
                                                 int g, float* sQ, const float* sG, Sink sink) {
  constexpr int ROWS = 16 * NQ, C = D / 16, F = D / 64, OST = D + 4;
  constexpr int SPLIT = WAVES / (2 * F), NP = (NQ + SPLIT - 1) / SPLIT;   // wavefronts that share the rows; sixteens of rows of one
  __shared__ float gpart[ROWS][2 * F], dpart[ROWS][WAVES];
  const float* bq0 = sQ + l16 * OST + 4 * g;
  const float* bg0 = sG + l16 * OST + 4 * g;
  // Wavefront kz computes, for its rows, the value features (of num) and key features (of the gradient) 64 f + 4 i + 2 pr and
  // + 1: one rotation pair in one lane
  const float* L = hist.L + (size_t)bh * D * D;
  const float* z = hist.z + (size_t)bh * D;
  const T* qh = static_cast<const T*>(hist.q_hist);
#pragma unroll
  for (int n = 0; n < NQ; ++n) {   // every wavefront its share of the features: R(phi(q)) into Q's place, its part of phi(q).z
    const size_t qrow = (size_t)min(row0 + 16 * n + l16, n_q - 1);
    float acc = 0.0f;
#pragma unroll
    for (int u = 0; u < (C + WAVES - 1) / WAVES; ++u) {
      const int c = kz + WAVES * u;
      if (C % WAVES && c >= C) break;   // uniform
      f32x4 x = load4<T>(qh + ((size_t)bh * n_q + qrow) * D + 16 * c + 4 * g);
      const f32x4 zz = *reinterpret_cast<const f32x4*>(z + 16 * c + 4 * g);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        x[e] = phi_apply(x[e], hist.phi_kind);
        acc = fmaf(x[e], zz[e], acc);
      }
      if (hist.cosq) {
        const size_t at = qrow * (D / 2) + 8 * c + 2 * g;
        const f32x2 cs = *reinterpret_cast<const f32x2*>(hist.cosq + at), sn = *reinterpret_cast<const f32x2*>(hist.sinq + at);
        x = rotate4(x, cs[0], sn[0], cs[1], sn[1]);
      }
      *reinterpret_cast<f32x4*>(sQ + (16 * n + l16) * OST + 16 * c + 4 * g) = x;
    }
    acc = column_sum(acc);
    if (g == 0) dpart[16 * n + l16][kz] = acc;
  }
  __syncthreads();
  const int f0 = (kz >> 1) % F, pr = kz & 1, n0 = kz / (2 * F) * NP;
  const bool active = n0 < NQ;   // uniform
  float den[NP];
#pragma unroll
  for (int n = 0; n < NP; ++n) {
    float acc = 0.0f;
#pragma unroll
    for (int u = 0; u < (C < WAVES ? C : WAVES); ++u) acc += dpart[16 * min(n0 + n, NQ - 1) + l16][u];
    den[n] = 1.0f / (hist.z_scale * acc + hist.eps);   // (the reciprocal from here on)
  }
  if (active) {
    f32x4 num[NP][2];
#pragma unroll
    for (int n = 0; n < NP; ++n) num[n][0] = num[n][1] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 2
    for (int c = 0; c < C; ++c) {
      f32x2 a[4];
#pragma unroll
      for (int r = 0; r < 4; ++r)
        a[r] = *reinterpret_cast<const f32x2*>(L + (size_t)(16 * c + 4 * g + r) * D + 64 * f0 + 4 * l16 + 2 * pr);
#pragma unroll
      for (int n = 0; n < NP; ++n) {
        const f32x4 b = *reinterpret_cast<const f32x4*>(bq0 + 16 * (n0 + n) * OST + 16 * c);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          num[n][0] = mfma_f32(a[r][0], b[r], num[n][0]);
          num[n][1] = mfma_f32(a[r][1], b[r], num[n][1]);
        }
      }
    }
#pragma unroll
    for (int n = 0; n < NP; ++n) {
      float acc = 0.0f;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const f32x2 x = *reinterpret_cast<const f32x2*>(sG + (16 * (n0 + n) + l16) * OST + 64 * f0 + 16 * g + 4 * r + 2 * pr);
        acc = fmaf(num[n][0][r], x[0], fmaf(num[n][1][r], x[1], acc));
      }
      acc = column_sum(acc);
      if (g == 0) gpart[16 * (n0 + n) + l16][kz % (2 * F)] = acc;
    }
  }
  __syncthreads();
  if (active) {
    f32x4 tt[NP][2];
#pragma unroll
    for (int n = 0; n < NP; ++n) tt[n][0] = tt[n][1] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const float* La = L + (size_t)(64 * f0 + 4 * l16 + 2 * pr) * D + 4 * g;
#pragma unroll 2
    for (int c = 0; c < C; ++c) {
      const f32x4 a0 = *reinterpret_cast<const f32x4*>(La + 16 * c), a1 = *reinterpret_cast<const f32x4*>(La + D + 16 * c);
#pragma unroll
      for (int n = 0; n < NP; ++n) {
        const f32x4 b = *reinterpret_cast<const f32x4*>(bg0 + 16 * (n0 + n) * OST + 16 * c);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          tt[n][0] = mfma_f32(a0[e], b[e], tt[n][0]);
          tt[n][1] = mfma_f32(a1[e], b[e], tt[n][1]);
        }
      }
    }
#pragma unroll
    for (int n = 0; n < NP; ++n) {
      const int rr = row0 + 16 * (n0 + n) + l16;
      const size_t qrow = (size_t)min(rr, n_q - 1);
      float gn = 0.0f;
#pragma unroll
      for (int u = 0; u < 2 * F; ++u) gn += gpart[16 * (n0 + n) + l16][u];
      const float dden = -gn * den[n] * den[n] * hist.z_scale;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int feat = 64 * f0 + 16 * g + 4 * r + 2 * pr;
        float t0 = tt[n][0][r] * den[n], t1 = tt[n][1][r] * den[n];
        if (hist.cosq) {   // the opposite angle
          const float cs = hist.cosq[qrow * (D / 2) + feat / 2], sn = hist.sinq[qrow * (D / 2) + feat / 2];
          const float u0 = t0 * cs + t1 * sn;
          t1 = t1 * cs - t0 * sn;
          t0 = u0;
        }
        const T* qp = qh + ((size_t)bh * n_q + qrow) * D + feat;
        const float q0 = Elem<T>::load(qp), q1 = Elem<T>::load(qp + 1);
        const bool relu = hist.phi_kind == HF_PHI_RELU;
        const float d0 = q0 > 0.0f ? 1.0f : (relu ? 0.0f : __expf(q0)), d1 = q1 > 0.0f ? 1.0f : (relu ? 0.0f : __expf(q1));
        const f32x2 zz = *reinterpret_cast<const f32x2*>(z + feat);
        const float v0 = fmaf(dden, zz[0], t0) * d0, v1 = fmaf(dden, zz[1], t1) * d1;
        if (hist.dq_hist) {
          if (rr < q_end) {
            T* dst = static_cast<T*>(hist.dq_hist) + ((size_t)bh * n_q + rr) * D + feat;
            Elem<T>::store(dst, v0);
            Elem<T>::store(dst + 1, v1);
          }
        } else {
          sink(n0 + n, f0, pr, r, v0, v1);
        }
      }
    }
  }
}

// ---- dQ: a workgroup per 16 NQ query rows; S^T and dP^T = V dO^T (row form), dS^T = P^T (dP^T - D), dQ^T += K^T dS^T
// (column form), all on 16 x 16 x 4 fp32 products.  Q and dO wait in LDS (B operands, shared by the four wavefronts); the
// keys' and values' pieces travel one product phase ahead, each into the registers of a piece that has just been used.
// kStored: S and dP come from bwd_scores_kernel, the products are dQ's alone.  Bound by the fp32 matrix rate.  12 heads of
// 128, 1170 x 2340, k = 10 of 37 blocks of 64, on its own: 88 us (0.71 ms with one key per lane and FMA arithmetic, plus
// 0.21 ms for the history branch's gradient as a kernel of its own).
template <typename T, int D, int NQ, bool kStored>
__device__ __forceinline__ void dq_role(const WideBwd& a, int wg, float* __restrict__ smem) {
  // with stored scores the wavefronts split a head's features as well as the list
  constexpr int ROWS = 16 * NQ, F = D / 64, OST = D + 4, WAVES = kStored ? kStoredWaves : kParts, FW = kStored ? 1 : F;
  constexpr int PARTS = WAVES * FW / F, AT_ONCE = kStored ? 2 : PARTS;
  float* sQ = smem;                 // [ROWS][OST] Q, [ROWS][OST] dO; later partial results
  float* sG = smem + ROWS * OST;
  const T* __restrict__ Q = static_cast<const T*>(a.Q);
  const T* __restrict__ dO = static_cast<const T*>(a.dO);
  const int k = a.k, n_q = a.n_q, n_kv = a.n_kv, bq = a.bq, bkv = a.bkv, t_m = a.t_m, t_n = a.t_n;
  const WideBwdHist& hist = a.hist;
  const int item = (wg & 7) * a.q_per_xcd + (wg >> 3);
  if ((wg >> 3) >= a.q_per_xcd || item >= a.q_total) return;
  const int bh = item / (t_m * a.q_chunks), in_head = item - bh * t_m * a.q_chunks;
  const int qb = in_head / a.q_chunks, row0 = qb * bq + (in_head - qb * a.q_chunks) * ROWS;
  const int q_end = min(n_q, (qb + 1) * bq);
  if (row0 >= q_end) return;
  const int lane = threadIdx.x & 63, kz = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  const int part = kz % PARTS, f_own = kz / PARTS;   // (f_own: the first of the wavefront's FW pieces of 64 features)
  const T* __restrict__ Kh = static_cast<const T*>(a.K) + (size_t)bh * a.kv_stride * D;
  const T* __restrict__ Vh = static_cast<const T*>(a.V) + (size_t)bh * a.kv_stride * D;
  const int32_t* __restrict__ row_idx = a.idx ? a.idx + ((size_t)bh * t_m + qb) * k : nullptr;
  const int nsel = a.idx ? k : t_n, subs = (bkv + 15) / 16, ntiles = nsel * subs;

  if (!kStored || hist.L)   // (uniform; with stored scores only the history branch reads them)
    for (int e = threadIdx.x; e < ROWS * (D / 4); e += 64 * WAVES) {
      const int rr = e / (D / 4), c4 = e - rr * (D / 4);
      const size_t off = ((size_t)bh * n_q + min(row0 + rr, n_q - 1)) * D + 4 * c4;
      if (!kStored) *reinterpret_cast<f32x4*>(sQ + rr * OST + 4 * c4) = load4<T>(Q + off) * a.scale_log2e;
      *reinterpret_cast<f32x4*>(sG + rr * OST + 4 * c4) = load4<T>(dO + off);
    }
  __syncthreads();

  float lse[NQ], dv[NQ];
  f32x4 dq[NQ][FW][4];
#pragma unroll
  for (int n = 0; n < NQ; ++n) {
    const size_t at = (size_t)bh * n_q + min(row0 + 16 * n + l16, n_q - 1);
    lse[n] = a.lse2[at];
    dv[n] = a.Dv[at];
  }
  auto zero = [&]() {
#pragma unroll
    for (int n = 0; n < NQ; ++n)
#pragma unroll
      for (int f = 0; f < FW; ++f)
#pragma unroll
        for (int e = 0; e < 4; ++e) dq[n][f][e] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  };
  auto tile_at = [&](int t, int& first, int& cnt) {   // cnt 0: past the list, an index out of range, or no such keys
    const int s = t / subs, sub = t - s * subs;
    // (no branch, which in the loop would have the accumulators kept twice: a dense window has some word read in its place)
    const int e = (row_idx ? row_idx : reinterpret_cast<const int32_t*>(a.lse2))[row_idx ? min(s, nsel - 1) : 0];
    const int jb = row_idx ? e : s;
    const int st = jb * bkv + 16 * sub;
    const bool ok = s < nsel && (unsigned)jb < (unsigned)t_n;
    const int n = ok ? min(16, min(n_kv, (jb + 1) * bkv) - st) : 0;
    cnt = n > 0 ? n : 0;
    first = n > 0 ? st : 0;
  };
  if constexpr (kStored) {
    if (hist.L) {   // first, into Q's place, while the accumulators' registers are free
      history_gradient<T, D, NQ, WAVES>(hist, bh, row0, q_end, n_q, kz, l16, g, sQ, sG, [&](int n, int f, int pr, int r, float v0, float v1) {
        *reinterpret_cast<f32x2*>(sQ + (16 * n + l16) * OST + 64 * f + 16 * g + 4 * r + 2 * pr) = f32x2{v0, v1};
      });
      __syncthreads();
    }
    zero();
    // S and dP of a tile lie where bwd_scores_kernel left them, four keys of a query to a lane: what the B operand takes.
    const int qt = (bq + 15) / 16, qi0 = (row0 - qb * bq) / 16;
    constexpr int B = sizeof(T);
    int col_at = (4 * g * D + 64 * f_own + 4 * l16) * B, tile_lane = (16 * l16 + 4 * g) * 4;
    Piece<T> kc[4];
    f32x4 s[NQ], p[NQ];
    auto request_scores = [&](int t, int cnt) {
      const int slot = t / subs, sub = t - slot * subs;
#pragma unroll
      for (int n = 0; n < NQ; ++n) {
        const float* tile = score_tile(a, bh, qb, min(slot, nsel - 1), min(qi0 + n, qt - 1), sub);
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(tile), 0, cnt > 0 ? kScoreTile * 4 : 0, 0x00020000);
        s[n] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, tile_lane, 0, 0));
        p[n] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, tile_lane + kScoreTile * 2, 0, 0));
      }
    };
    int first, cnt;
    tile_at(part, first, cnt);
    request_scores(part, __builtin_amdgcn_readfirstlane(cnt));
    const __amdgpu_buffer_rsrc_t k_rows = tile_rows<T, D>(Kh, first, cnt);
#pragma unroll
    for (int u = 0; u < 4; ++u) kc[u].load(k_rows, col_at + u * D * B);
    for (int t = part; t < ntiles; t += PARTS) {
      asm volatile("" : "+v"(col_at), "+v"(tile_lane));   // (opaque here, or their sums leave the loop as registers instead of immediates)
      f32x4 ds[NQ];   // zero for a key that does not exist: its S is -inf, or the tile has none
#pragma unroll
      for (int n = 0; n < NQ; ++n) {
        const float off = cnt > 0 ? lse[n] : __builtin_inff();
#pragma unroll
        for (int r = 0; r < 4; ++r) ds[n][r] = __builtin_amdgcn_exp2f(s[n][r] - off) * (p[n][r] - dv[n]);
      }
      tile_at(t + PARTS, first, cnt);
      const __amdgpu_buffer_rsrc_t kn_rows = tile_rows<T, D>(Kh, first, cnt);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (u == 2) request_scores(t + PARTS, __builtin_amdgcn_readfirstlane(cnt));
        const f32x4 ka = kc[u].get();
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int n = 0; n < NQ; ++n) dq[n][0][e] = mfma_f32(ka[e], ds[n][u], dq[n][0][e]);
        kc[u].load(kn_rows, col_at + u * D * B);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  } else {
    zero();
    const float* bq0 = sQ + l16 * OST + 4 * g;
    const float* bg0 = sG + l16 * OST + 4 * g;
    constexpr int C = D / 16;
    Piece<T> kr[C], vr[C], kc[4][F];
    int first, cnt, first_n, cnt_n;
    tile_at(kz, first, cnt);
    constexpr int B = sizeof(T);
    int row_at = (l16 * D + 4 * g) * B, col_at = (4 * g * D + 4 * l16) * B;   // rows behind a tile's last real key read as zeros
    __amdgpu_buffer_rsrc_t k_rows = tile_rows<T, D>(Kh, first, cnt);
    {
      const __amdgpu_buffer_rsrc_t v_rows = tile_rows<T, D>(Vh, first, cnt);
#pragma unroll
      for (int c = 0; c < C; ++c) {
        kr[c].load(k_rows, row_at + 16 * c * B);
        vr[c].load(v_rows, row_at + 16 * c * B);
        __builtin_amdgcn_sched_barrier(0);   // (requests are awaited in order: in this order here and in the loop)
      }
    }
    for (int t = kz; t < ntiles; t += kParts) {
      asm volatile("" : "+v"(row_at), "+v"(col_at));   // (opaque here, or their sums leave the loop as registers instead of immediates)
      tile_at(t + kParts, first_n, cnt_n);
      const __amdgpu_buffer_rsrc_t kn_rows = tile_rows<T, D>(Kh, first_n, cnt_n), vn_rows = tile_rows<T, D>(Vh, first_n, cnt_n);
      f32x4 s[NQ], p[NQ];
#pragma unroll
      for (int n = 0; n < NQ; ++n) s[n] = p[n] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int c = 0; c < C; ++c) {
        const f32x4 a = kr[c].get(), v = vr[c].get();
        f32x4 b[NQ], gg[NQ];
#pragma unroll
        for (int n = 0; n < NQ; ++n) {
          b[n] = *reinterpret_cast<const f32x4*>(bq0 + 16 * n * OST + 16 * c);
          gg[n] = *reinterpret_cast<const f32x4*>(bg0 + 16 * n * OST + 16 * c);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int n = 0; n < NQ; ++n) {
            s[n] = mfma_f32(a[e], b[n][e], s[n]);
            p[n] = mfma_f32(v[e], gg[n][e], p[n]);
          }
#pragma unroll
        for (int u = c * 4 * F / C; u < (c + 1) * 4 * F / C; ++u) kc[u / F][u % F].load(k_rows, col_at + (u / F * D + 64 * (u % F)) * B);
        __builtin_amdgcn_sched_barrier(0);
      }
      // dS = P (dP - D); zero for a key that does not exist
#pragma unroll
      for (int n = 0; n < NQ; ++n)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float ds = __builtin_amdgcn_exp2f(s[n][r] - lse[n]) * (p[n][r] - dv[n]);
          s[n][r] = 4 * g + r < cnt ? ds : 0.0f;
        }
#pragma unroll
      for (int u = 0; u < 4 * F; ++u) {
        const f32x4 a = kc[u / F][u % F].get();
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int n = 0; n < NQ; ++n) dq[n][u % F][e] = mfma_f32(a[e], s[n][u / F], dq[n][u % F][e]);
#pragma unroll
        for (int c = u * C / (4 * F); c < (u + 1) * C / (4 * F); ++c) {
          kr[c].load(kn_rows, row_at + 16 * c * B);
          vr[c].load(vn_rows, row_at + 16 * c * B);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      k_rows = kn_rows;
      cnt = cnt_n;
    }
  }
#pragma unroll
  for (int n = 0; n < NQ; ++n)
#pragma unroll
    for (int f = 0; f < FW; ++f)
#pragma unroll
      for (int e = 0; e < 4; ++e) dq[n][f][e] *= a.scale;
  __syncthreads();   // Q and dO are read no more as operands of the loop

  if constexpr (!kStored) {
    if (hist.L) {
      history_gradient<T, D, NQ, WAVES>(hist, bh, row0, q_end, n_q, kz, l16, g, sQ, sG, [&](int n, int f0, int pr, int r, float v0, float v1) {
#pragma unroll
        for (int m = 0; m < NQ; ++m)   // (constant indices into the accumulators)
#pragma unroll
          for (int f = 0; f < FW; ++f)
#pragma unroll
            for (int q = 0; q < 2; ++q)
              if (m == n && f == f0 && q == pr) {
                dq[m][f][2 * q][r] += v0;
                dq[m][f][2 * q + 1][r] += v1;
              }
      });
      __syncthreads();
    }
  }
  add_parts<D, NQ, PARTS, AT_ONCE, FW>(smem, dq, 1.0f, kStored && hist.L && !hist.dq_hist, part, f_own, l16, g);
  store_parts<T, D, NQ, AT_ONCE, WAVES>(smem, static_cast<T*>(a.dQ) + ((size_t)bh * n_q + row0) * D, q_end - row0, threadIdx.x);
}

// ---- dK, dV: a workgroup per 16 NK keys of a KV block, its four wavefronts taking every fourth 16-row tile of the query
// blocks on the inverse list.  S = Q K^T, dP = dO V^T (row form; K and V wait in LDS), P = 2^(S - lse2), dS = P (dP - D),
// dV^T += dO^T P, dK^T += Q^T dS (column form).  Bound by the fp32 matrix rate, at the same shape 118 us (1.01 ms with one
// query per lane and FMA arithmetic).
template <typename T, int D, int NK>
__device__ __forceinline__ void dkv_role(const WideBwd& a, int wg, float* __restrict__ smem) {
  constexpr int ROWS = 16 * NK, C = D / 16, F = D / 64, OST = D + 4;
  float* sK = smem;                 // [ROWS][OST] K, [ROWS][OST] V; later four partial results
  float* sV = smem + ROWS * OST;
  const T* __restrict__ K = static_cast<const T*>(a.K);
  const T* __restrict__ V = static_cast<const T*>(a.V);
  const int n_q = a.n_q, n_kv = a.n_kv, kv_stride = a.kv_stride, bq = a.bq, bkv = a.bkv, t_m = a.t_m, t_n = a.t_n;
  const int item = (wg & 7) * a.k_per_xcd + (wg >> 3);
  if ((wg >> 3) >= a.k_per_xcd || item >= a.k_total) return;
  const int bh = item / (t_n * a.k_chunks), in_head = item - bh * t_n * a.k_chunks;
  const int jb = in_head / a.k_chunks, key0 = jb * bkv + (in_head - jb * a.k_chunks) * ROWS;
  const int k_end = min(n_kv, (jb + 1) * bkv);
  if (key0 >= k_end) return;
  const int lane = threadIdx.x & 63, kz = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  const T* __restrict__ Qh = static_cast<const T*>(a.Q) + (size_t)bh * n_q * D;
  const T* __restrict__ Gh = static_cast<const T*>(a.dO) + (size_t)bh * n_q * D;
  const float* __restrict__ lseh = a.lse2 + (size_t)bh * n_q;
  const float* __restrict__ dvh = a.Dv + (size_t)bh * n_q;
  const int n_lists = a.inv_cnt ? a.inv_cnt[(size_t)bh * t_n + jb] : t_m;   // no lists: every query block (dense)
  const int32_t* __restrict__ list = a.inv_list ? a.inv_list + ((size_t)bh * t_n + jb) * t_m : nullptr;
  const int subs = (bq + 15) / 16, ntiles = n_lists * subs;

  f32x4 ak[NK][F][4], av[NK][F][4];
#pragma unroll
  for (int n = 0; n < NK; ++n)
#pragma unroll
    for (int f = 0; f < F; ++f)
#pragma unroll
      for (int e = 0; e < 4; ++e) ak[n][f][e] = av[n][f][e] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  for (int e = threadIdx.x; e < ROWS * (D / 4); e += 64 * kParts) {
    const int rr = e / (D / 4), c4 = e - rr * (D / 4);
    const size_t off = ((size_t)bh * kv_stride + min(key0 + rr, n_kv - 1)) * D + 4 * c4;
    *reinterpret_cast<f32x4*>(sK + rr * OST + 4 * c4) = load4<T>(K + off) * a.scale_log2e;
    *reinterpret_cast<f32x4*>(sV + rr * OST + 4 * c4) = load4<T>(V + off);
  }
  __syncthreads();

  auto tile_at = [&](int t, int& first, int& cnt) {   // cnt 0: past the list or past the last query
    const int s = t / subs, sub = t - s * subs;
    const int qb = s < n_lists ? (list ? list[s] : s) : 0;
    const int st = qb * bq + 16 * sub;
    const int n = s < n_lists ? min(16, min(n_q, (qb + 1) * bq) - st) : 0;
    cnt = n > 0 ? n : 0;
    first = n > 0 ? st : 0;
  };
  Piece<T> qr[C], gr[C], qc[4][F], gc[4][F];
  int first, cnt, first_n, cnt_n;
  tile_at(kz, first, cnt);
  constexpr int B = sizeof(T);
  int row_at = (l16 * D + 4 * g) * B, col_at = (4 * g * D + 4 * l16) * B;   // rows behind a tile's last real query read as zeros
  __amdgpu_buffer_rsrc_t q_rows = tile_rows<T, D>(Qh, first, cnt), g_rows = tile_rows<T, D>(Gh, first, cnt);
#pragma unroll
  for (int c = 0; c < C; ++c) {
    qr[c].load(q_rows, row_at + 16 * c * B);
    gr[c].load(g_rows, row_at + 16 * c * B);
    __builtin_amdgcn_sched_barrier(0);
  }
  const float* bk0 = sK + l16 * OST + 4 * g;
  const float* bv0 = sV + l16 * OST + 4 * g;
  for (int t = kz; t < ntiles; t += kParts) {
    asm volatile("" : "+v"(row_at), "+v"(col_at));   // (opaque here, or their sums leave the loop as registers instead of immediates)
    tile_at(t + kParts, first_n, cnt_n);
    const __amdgpu_buffer_rsrc_t qn_rows = tile_rows<T, D>(Qh, first_n, cnt_n), gn_rows = tile_rows<T, D>(Gh, first_n, cnt_n);
    float lse[4], dv[4];   // (of the tile's last query for those that do not exist: what they give is dropped)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = __builtin_amdgcn_readfirstlane(first) + min(4 * g + r, max(cnt - 1, 0));
      lse[r] = lseh[row];
      dv[r] = dvh[row];
    }
    f32x4 s[NK], p[NK];
#pragma unroll
    for (int n = 0; n < NK; ++n) s[n] = p[n] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const f32x4 a = qr[c].get(), v = gr[c].get();
      f32x4 b[NK], gg[NK];
#pragma unroll
      for (int n = 0; n < NK; ++n) {
        b[n] = *reinterpret_cast<const f32x4*>(bk0 + 16 * n * OST + 16 * c);
        gg[n] = *reinterpret_cast<const f32x4*>(bv0 + 16 * n * OST + 16 * c);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int n = 0; n < NK; ++n) {
          s[n] = mfma_f32(a[e], b[n][e], s[n]);
          p[n] = mfma_f32(v[e], gg[n][e], p[n]);
        }
#pragma unroll
      for (int u = c * 4 * F / C; u < (c + 1) * 4 * F / C; ++u) {
        gc[u / F][u % F].load(g_rows, col_at + (u / F * D + 64 * (u % F)) * B);
        qc[u / F][u % F].load(q_rows, col_at + (u / F * D + 64 * (u % F)) * B);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    // P and dS; zero for a query that does not exist
#pragma unroll
    for (int n = 0; n < NK; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const bool real = 4 * g + r < cnt;
        const float w = __builtin_amdgcn_exp2f(s[n][r] - lse[r]), ds = w * (p[n][r] - dv[r]);
        s[n][r] = real ? w : 0.0f;
        p[n][r] = real ? ds : 0.0f;
      }
#pragma unroll
    for (int u = 0; u < 4 * F; ++u) {
      const f32x4 a = gc[u / F][u % F].get(), b = qc[u / F][u % F].get();
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int n = 0; n < NK; ++n) {
          av[n][u % F][e] = mfma_f32(a[e], s[n][u / F], av[n][u % F][e]);
          ak[n][u % F][e] = mfma_f32(b[e], p[n][u / F], ak[n][u % F][e]);
        }
#pragma unroll
      for (int c = u * C / (4 * F); c < (u + 1) * C / (4 * F); ++c) {
        qr[c].load(qn_rows, row_at + 16 * c * B);
        gr[c].load(gn_rows, row_at + 16 * c * B);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    first = first_n;
    q_rows = qn_rows;
    g_rows = gn_rows;
    cnt = cnt_n;
  }
  __syncthreads();   // K and V are read no more
  const size_t out = ((size_t)bh * kv_stride + key0) * D;
  add_parts<D, NK, kParts, kParts, F>(smem, ak, a.scale, false, kz, 0, l16, g);
  store_parts<T, D, NK, kParts, kParts>(smem, static_cast<T*>(a.dK) + out, k_end - key0, threadIdx.x);
  __syncthreads();
  add_parts<D, NK, kParts, kParts, F>(smem, av, 1.0f, false, kz, 0, l16, g);
  store_parts<T, D, NK, kParts, kParts>(smem, static_cast<T*>(a.dV) + out, k_end - key0, threadIdx.x);
}

// ---- dK, dV from stored scores: a workgroup per 16 NK keys of a KV block, half of its wavefronts for each of the two (half of the
// accumulators a wavefront: four of them on a SIMD).
template <typename T, int D, int NK>
__device__ __forceinline__ void dkv_stored_role(const WideBwd& a, int wg, float* __restrict__ smem) {
  constexpr int ROWS = 16 * NK, F = D / 64, OST = D + 4;
  constexpr bool kTight = NK * F == 4;   // all 128 registers are in use: the loop keeps one for what a lane's four queries follow from
  const int n_q = a.n_q, n_kv = a.n_kv, kv_stride = a.kv_stride, bq = a.bq, bkv = a.bkv, t_m = a.t_m, t_n = a.t_n;
  const int place = wg >> 3, chunk = place % a.k_chunks, block = (wg & 7) * (a.k_per_xcd / a.k_chunks) + place / a.k_chunks;
  if (place >= a.k_per_xcd || block >= a.k_total / a.k_chunks) return;
  const int32_t* rec = a.order ? a.order + (size_t)block * kOrderRec : nullptr;
  const int item = rec ? rec[0] : block, bh = item / t_n, jb = item - bh * t_n, key0 = jb * bkv + chunk * ROWS;
  const int k_end = min(n_kv, (jb + 1) * bkv);
  if (key0 >= k_end) return;
  const int lane = threadIdx.x & 63, kz = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  constexpr int PARTS = kStoredWaves / 2;
  const int part = kz % PARTS;
  const bool keys = kz >= PARTS;     // the first half: dV^T += dO^T P; the second: dK^T += Q^T dS
  const T* __restrict__ Xh = static_cast<const T*>(keys ? a.Q : a.dO) + (size_t)bh * n_q * D;
  const float* __restrict__ lseh = a.lse2 + (size_t)bh * n_q;
  const float* __restrict__ dvh = a.Dv + (size_t)bh * n_q;
  const int n_lists = rec ? rec[1] : a.inv_cnt ? a.inv_cnt[item] : t_m;   // no lists: every query block (dense)
  const int32_t* __restrict__ list = a.inv_list ? a.inv_list + ((size_t)bh * t_n + jb) * t_m : nullptr;
  const int subs = (bq + 15) / 16, ntiles = n_lists * subs;

  f32x4 acc[NK][F][4];
#pragma unroll
  for (int n = 0; n < NK; ++n)
#pragma unroll
    for (int f = 0; f < F; ++f)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[n][f][e] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  const int32_t* __restrict__ slots = a.inv_slot ? a.inv_slot + ((size_t)bh * t_n + jb) * t_m : nullptr;
  const int kt = (bkv + 15) / 16, ki0 = (key0 - jb * bkv) / 16;
  constexpr int B = sizeof(T);
  int col_at = (4 * g * D + 4 * l16) * B, tile_lane = (64 * g + l16) * 4, g16 = 16 * g;
  // the list's entries are read a trip before their tile's rows are asked for (without a branch, which in the loop would
  // have the accumulators kept twice; a dense window has some word read in their place)
  const int32_t* __restrict__ some = reinterpret_cast<const int32_t*>(lseh);
  auto entry = [&](int t, int& qb, int& slot) {
    const int at = min(t / subs, max(n_lists - 1, 0)), from = list ? at : 0;
    const int b = (list ? list : some)[from], sl = (list ? slots : some)[from];
    qb = list ? b : at;
    slot = list ? sl : jb;
  };
  auto tile_of = [&](int t, int qb, int& first, int& cnt) {   // cnt 0: past the list or past the last query
    const int st = qb * bq + 16 * (t % subs);
    const int n = t < ntiles ? min(16, min(n_q, (qb + 1) * bq) - st) : 0;
    cnt = n > 0 ? n : 0;
    first = n > 0 ? st : 0;
  };
  // (half of a tile's pieces at a time: with a whole tile's the registers of four workgroups a compute unit do not suffice)
  constexpr int AHEAD = 2 * F;
  Piece<T> xc[AHEAD];
  float s[NK][4], p[NK][4], lse[4], dv[4];
  auto request_scores = [&](int t, int qb, int slot, int first, int cnt) {
    const __amdgpu_buffer_rsrc_t rl = tile_rows<float, 1>(lseh, first, cnt), rd = tile_rows<float, 1>(dvh, first, cnt);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      lse[r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rl, (kTight ? g16 : 16 * g) + 4 * r, 0, 0));
      dv[r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rd, (kTight ? g16 : 16 * g) + 4 * r, 0, 0));
    }
#pragma unroll
    for (int n = 0; n < NK; ++n) {
      const float* tile = score_tile(a, bh, qb, slot, t % subs, min(ki0 + n, kt - 1));
      // (dV takes S alone: what lies behind it reads as zeros, without a request to memory)
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<float*>(tile), 0, cnt > 0 ? kScoreTile * (keys ? 4 : 2) : 0, 0x00020000);
#pragma unroll
      for (int r = 0; r < 4; ++r) {   // a key to a lane, four queries: what the B operands take
        s[n][r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, tile_lane + 64 * r, 0, 0));
        p[n][r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, tile_lane + 64 * r + kScoreTile * 2, 0, 0));
      }
    }
  };
  int first, cnt, qb, slot, qb_n, slot_n;
  entry(part, qb, slot);
  entry(part + PARTS, qb_n, slot_n);
  tile_of(part, qb, first, cnt);
  request_scores(part, qb, slot, first, cnt);
  __amdgpu_buffer_rsrc_t x_rows = tile_rows<T, D>(Xh, first, cnt);
#pragma unroll
  for (int u = 0; u < AHEAD; ++u) xc[u].load(x_rows, col_at + (u / F * D + 64 * (u % F)) * B);
  for (int t = part; t < ntiles; t += PARTS) {
    if constexpr (kTight) asm volatile("" : "+v"(g16));
    asm volatile("" : "+v"(col_at), "+v"(tile_lane));   // (opaque here, or their sums leave the loop as registers instead of immediates)
    float w[NK][4];   // P (P (0 + 1)) or dS = P (dP - D)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const bool real = kTight ? g16 < 4 * (cnt - r) : 4 * g + r < cnt;
      const float off = keys ? dv[r] : -1.0f;
#pragma unroll
      for (int n = 0; n < NK; ++n) {
        const float v = __builtin_amdgcn_exp2f(s[n][r] - lse[r]) * (p[n][r] - off);
        w[n][r] = real ? v : 0.0f;   // zero for a query that does not exist
      }
    }
    int first_n, cnt_n;
    tile_of(t + PARTS, qb_n, first_n, cnt_n);
    const __amdgpu_buffer_rsrc_t xn_rows = tile_rows<T, D>(Xh, first_n, cnt_n);
#pragma unroll
    for (int u = 0; u < 4 * F; ++u) {
      if (u == 3 * F) {   // (three quarters of the weights are used up: their registers take the next tile's)
        request_scores(t + PARTS, qb_n, slot_n, first_n, cnt_n);
        entry(t + 2 * PARTS, qb_n, slot_n);
      }
      const f32x4 xa = xc[u % AHEAD].get();
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int n = 0; n < NK; ++n) acc[n][u % F][e] = mfma_f32(xa[e], w[n][u / F], acc[n][u % F][e]);
      const int v = (u + AHEAD) % (4 * F), at = col_at + (v / F * D + 64 * (v % F)) * B;
      xc[u % AHEAD].load(u < AHEAD ? x_rows : xn_rows, at);
      __builtin_amdgcn_sched_barrier(0);
    }
    cnt = cnt_n;
    x_rows = xn_rows;
  }
  float* const own = smem + (keys ? 2 * ROWS * OST : 0);
  int tid = threadIdx.x, l_end = l16, g_end = g;
  if constexpr (kTight) {   // (formed again instead of kept over the loop)
    const int again = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    tid = 64 * kz + again;
    l_end = again & 15;
    g_end = again >> 4;
  }
  add_parts<D, NK, PARTS, 2, F>(own, acc, keys ? a.scale : 1.0f, false, part, 0, l_end, g_end);
  const size_t out = ((size_t)bh * kv_stride + key0) * D;
  store_parts<T, D, NK, 2, kStoredWaves>(smem, static_cast<T*>(a.dV) + out, k_end - key0, tid);
  store_parts<T, D, NK, 2, kStoredWaves>(smem + 2 * ROWS * OST, static_cast<T*>(a.dK) + out, k_end - key0, tid);
}

template <typename T, int D, int NQ>
__global__ __launch_bounds__(64 * kParts, 2) void bwd_dq_wide_kernel(WideBwd a) {
  extern __shared__ __attribute__((aligned(16))) float smem[];
  dq_role<T, D, NQ, false>(a, blockIdx.x, smem);
}
template <typename T, int D, int NK>
__global__ __launch_bounds__(64 * kParts, 2) void bwd_dkv_wide_kernel(WideBwd a) {
  extern __shared__ __attribute__((aligned(16))) float smem[];
  dkv_role<T, D, NK>(a, blockIdx.x, smem);
}
// From stored scores, dQ's workgroups and behind them dK and dV's, longest list first, in one launch: bound by the fp32 matrix
// rate and by how evenly the last workgroups end.  At the sizes of bwd_scores_kernel 112 us with dK and dV in index order in
// front and two workgroups of four wavefronts a compute unit, 105 with dQ in front, 96..103 ordered, 98 with eight wavefronts a
// workgroup (half the chain each).  Scores and rows read from one place of the caches instead of their own: no faster.
template <typename T, int D, int NQ, int NK>
__global__ __launch_bounds__(64 * kStoredWaves, 4) void bwd_stored_kernel(WideBwd a) {
  extern __shared__ __attribute__((aligned(16))) float smem[];
  const int q_wgs = 8 * a.q_per_xcd;
  if ((int)blockIdx.x < q_wgs)
    dq_role<T, D, NQ, true>(a, blockIdx.x, smem);
  else
    dkv_stored_role<T, D, NK>(a, blockIdx.x - q_wgs, smem);
}

template <int D>
int launch_wide(const void* fn, LdsGrant& grant, long long wgs, int waves, int rows, WideBwd& a, hipStream_t s) {
  const int lds = rows * (D + 4) * (int)sizeof(float);
  if (lds > 64 * 1024) {
    const int rc = grant_lds(grant, fn, lds, "the fp32 backward kernels");
    if (rc != HF_OK) return rc;
  }
  void* args[] = {&a};
  (void)hipLaunchKernel(fn, dim3((unsigned)wgs), dim3(64 * waves), args, lds, s);
  return check_launch("hf_hybrid_attn_bwd(dQ, dK, dV)");
}

template <typename T, int D, int NQ, int NK>
int launch_bwd_wide(WideBwd& a, hipStream_t s) {
  static LdsGrant grants[4];
  constexpr int N = NQ > NK ? NQ : NK;
  const long long q_wgs = 8ll * a.q_per_xcd, k_wgs = 8ll * a.k_per_xcd;
  int rc;
  if (a.scores) {
    if ((rc = launch_wide<D>(reinterpret_cast<const void*>(bwd_scores_kernel<T, D, NQ>), grants[0], q_wgs, kScoreParts, 2 * 16 * NQ, a, s)) != HF_OK) return rc;
    return launch_wide<D>(reinterpret_cast<const void*>(bwd_stored_kernel<T, D, NQ, NK>), grants[1], q_wgs + k_wgs, kStoredWaves, 4 * 16 * N, a, s);
  }
  if ((rc = launch_wide<D>(reinterpret_cast<const void*>(bwd_dq_wide_kernel<T, D, NQ>), grants[2], q_wgs, kParts, kParts * 16 * NQ, a, s)) != HF_OK) return rc;
  return launch_wide<D>(reinterpret_cast<const void*>(bwd_dkv_wide_kernel<T, D, NK>), grants[3], k_wgs, kParts, kParts * 16 * NK, a, s);
}

}  // namespace

// idx given: the inverse lists (inv_slot given: with places), and with order given the launch order of the dK/dV
// items, `slabs` to a KV block; state given: planes (bf16, head_dim 128);
// A given: row dots (likewise).
int launch_bwd_prep(const hf_config& c, const int32_t* idx, int k, int t_m, int t_n, int32_t* inv_cnt, int32_t* inv_list,
                    int32_t* inv_slot, int32_t* order, int slabs, const float* state, void* planes, const void* A, const void* B, long long rows,
                    float* dots, hipStream_t s) {
  constexpr size_t kPrepLds = 150 * 1024;   // granted to the kernel below
  const int BH = c.batch * c.heads;
  PrepArgs p = {};
  p.idx = idx;
  p.k = k;
  p.t_m = t_m;
  p.t_n = t_n;
  p.inv_cnt = inv_cnt;
  p.inv_list = inv_list;
  p.inv_slot = inv_slot;
  size_t lds = 0;
  bool order_behind = false;
  const long long items = (long long)BH * t_n * slabs, share = (items + 7) / 8;
  if (order && items > (1ll << 29)) { set_error("too many blocks"); return HF_ERR_SHAPE; }
  if (idx) {
    const size_t words = ((size_t)t_m + 31) / 32, masks = (size_t)t_n * words * 4;
    const size_t need = ((size_t)share + t_m + 1 + ((size_t)share / slabs + 2) * words) * 4;
    // (the masks of a head in LDS, and a division by k in selected_by that is exact; the kernel of its own takes the rest:
    // 4 heads, 512 query and 1024 KV blocks, k = 256, 64 KB of masks: gradients 3.47 ms so, 4.54 through it in index order)
    if (masks <= kPrepLds && (unsigned long long)t_m * k * k < (1ull << 32)) {
      p.invert_wgs = BH;
      lds = masks;
      if (order && need <= kPrepLds) {
        p.order_wgs = 8;
        p.slabs = slabs;
        p.items_per_xcd = (int)share;
        p.total_items = (int)items;
        p.order = order;
        if (need > lds) lds = need;
      }
    } else {
      hipLaunchKernelGGL(invert_index_kernel, dim3((t_n + 3) / 4, BH), dim3(256), 0, s, idx, k, t_m, t_n, inv_cnt, inv_list,
                         inv_slot);
    }
    order_behind = order && !p.order_wgs;
  }
  if (state) {
    p.plane_wgs = 8 * BH;
    p.state = state;
    p.planes = static_cast<bf16_t*>(planes);
    if (lds < 2 * 32 * 33 * sizeof(float)) lds = 2 * 32 * 33 * sizeof(float);
  }
  long long dot_wgs = 0;
  if (A) {
    if (rows > (1ll << 34)) { set_error("too many rows"); return HF_ERR_SHAPE; }
    p.A = static_cast<const bf16_t*>(A);
    p.B = static_cast<const bf16_t*>(B);
    p.rows = rows;
    p.dots = dots;
    dot_wgs = (rows + kPrepThreads / 16 - 1) / (kPrepThreads / 16);
  }
  const long long wgs = p.order_wgs + p.invert_wgs + p.plane_wgs + dot_wgs;
  if (lds > 64 * 1024) {
    static LdsGrant grant;
    const int rc = grant_lds(grant, reinterpret_cast<const void*>(bwd_prep_kernel), (int)kPrepLds, "the backward pass's preparation");
    if (rc != HF_OK) return rc;
  }
  if (wgs) hipLaunchKernelGGL(bwd_prep_kernel, dim3((unsigned)wgs), dim3(kPrepThreads), lds, s, p);
  if (order_behind) {
    int shift = 0;
    while (t_m >> shift >= kLengths) ++shift;
    hipLaunchKernelGGL(dkv_order_kernel, dim3(8), dim3(kOrderThreads), 0, s, inv_cnt, inv_list, t_m, slabs, (int)share, (int)items,
                       shift, order);
  }
  return check_launch("hf_hybrid_attn_bwd(lists, planes, D)");
}

// Room for the stored scores, in a workspace of the size that callers are told.  It never shrinks as a call grows, so that one of the
// largest size serves the smaller ones, and ends at kScoresRoom: longer calls go through it a few heads at a time.
static size_t head_scores(const hf_config& c, int n_q, int k) {   // bytes of a head's
  const size_t t_m = (n_q + c.block_q - 1) / c.block_q, qt = (c.block_q + 15) / 16, kt = (c.block_kv + 15) / 16;
  return t_m * k * qt * kt * (kScoreTile * sizeof(float));
}

size_t bwd_scores_room(const hf_config& c, int n_q, int k) {
  const size_t all = (size_t)c.batch * c.heads * head_scores(c, n_q, k);
  return all < kScoresRoom ? all : kScoresRoom;
}

// 32 rows or keys a workgroup, 16 where a block has no more (or would leave over a quarter of the 32 empty): the second half of
// the products would be work on nothing
static int wide_rows(int block) { return (block + 31) / 32 * 32 * 3 <= block * 4 ? 32 : 16; }

// Heads whose scores are stored at a time, 0: none.  All that there is room for, in groups of a size, where the smallest has a
// query-side workgroup for every compute unit; with less, forming the products again for all heads at once is faster.  Products again /
// heads at a time, us: 12 heads of 128, 1170 x 2340, 38 workgroups a head: 244 / three 276, four 213, six 182, all 145; over every
// block 665 / three 709, four 537, all 452; 24 of 64, 1458 x 4374, half of the blocks, 46: 795 / three 910, four 756, eight 650, all
// 671; 12 of 64, 2000 x 4000, blocks of 128, 64: 283 / three 284, four 240, all 201; 12 of 128, 4680 x 9360, 148: 2410 / one 2433, two
// 2162, three 1832, all 1696; 24 of 64 in bf16, 148: 2643 / one 3137, two 2587, three 2119, twelve 1999.  Short blocks, whose tiles are
// padded to sixteen either way: 4 heads of 128, 64 x 128 in blocks of one 73 / all 50, 12, 600 x 600 in blocks of 4 749 / all 492.
int bwd_scores_heads(const hf_config& c, int n_q, int n_kv, int k, size_t room) {
  const size_t BH = (size_t)c.batch * c.heads, q_rows = wide_rows(c.block_q), k_rows = wide_rows(c.block_kv);
  const size_t q_wgs = (n_q + c.block_q - 1) / c.block_q * ((c.block_q + q_rows - 1) / q_rows);
  const size_t k_chunks = (c.block_kv + k_rows - 1) / k_rows, k_wgs = (n_kv + c.block_kv - 1) / c.block_kv * k_chunks;
  // (a launch has less than 2^32 threads, and both sides are rounded up to eight shares)
  const size_t most = (((size_t)1 << 32) / (64 * kStoredWaves) - 8 - 8 * k_chunks) / (q_wgs + k_wgs);
  const size_t fit = room / head_scores(c, n_q, k) < most ? room / head_scores(c, n_q, k) : most;
  if (fit >= BH) return (int)BH;
  return fit && BH / ((BH + fit - 1) / fit) * q_wgs >= 256 ? (int)fit : 0;
}

// dQ (with the history branch where a state, L and z, is given), dK and dV.
// scores given: room for them; NULL: lse2 and Dv are there already.
int launch_bwd_generic(const hf_config& c, const void* Q, const void* Q_hist, int n_q, const void* K, const void* V, int n_kv,
                       const int32_t* idx, int k, const void* dO, float* lse2, float* Dv, const int32_t* inv_cnt,
                       const int32_t* inv_list, const int32_t* inv_slot, const int32_t* order, float* scores, const float* state,
                       const float* zvec, const float* cosq, const float* sinq, void* dQ, void* dQ_hist, void* dK, void* dV, hipStream_t s) {
  WideBwd a = {};
  a.Q = Q; a.K = K; a.V = V; a.dO = dO;
  a.idx = idx;
  a.k = k; a.n_q = n_q; a.n_kv = n_kv;
  a.kv_stride = kv_stride_of(c, n_kv);
  a.bq = c.block_q; a.bkv = c.block_kv;
  a.t_m = (n_q + c.block_q - 1) / c.block_q;
  a.t_n = (n_kv + c.block_kv - 1) / c.block_kv;
  a.scale = c.softmax_scale > 0.0f ? c.softmax_scale : 1.0f / sqrtf((float)c.head_dim);
  a.scale_log2e = a.scale * 1.4426950408889634f;
  a.lse2 = lse2; a.Dv = Dv;
  a.inv_cnt = inv_cnt; a.inv_list = inv_list; a.inv_slot = inv_slot;
  a.order = order;
  a.scores = scores;
  a.dQ = dQ; a.dK = dK; a.dV = dV;
  if (state) {
    WideBwdHist& h = a.hist;
    h.L = state;
    h.z = zvec;
    h.cosq = cosq;
    h.sinq = sinq;
    h.q_hist = Q_hist;
    h.dq_hist = dQ_hist;
    h.eps = c.eps;
    h.z_scale = c.z_scale;
    h.phi_kind = c.phi;
  }
  const int q_rows = wide_rows(c.block_q), k_rows = wide_rows(c.block_kv);
  const bool q2 = q_rows == 32, k2 = k_rows == 32;
  a.q_chunks = (c.block_q + q_rows - 1) / q_rows;
  a.k_chunks = (c.block_kv + k_rows - 1) / k_rows;
  const long long BH = (long long)c.batch * c.heads, q_total = BH * a.t_m * a.q_chunks, k_total = BH * a.t_n * a.k_chunks;
  if (q_total > (1ll << 30) || k_total > (1ll << 30)) { set_error("too many blocks"); return HF_ERR_SHAPE; }
  a.q_total = (int)q_total;
  a.k_total = (int)k_total;
  a.q_per_xcd = (int)((q_total + 7) / 8);
  a.k_per_xcd = (int)((k_total / a.k_chunks + 7) / 8) * a.k_chunks;   // (whole blocks)
#define HF_BWD_WIDE(T, DD)                                                                     \
  return q2 ? (k2 ? launch_bwd_wide<T, DD, 2, 2>(a, s) : launch_bwd_wide<T, DD, 2, 1>(a, s))  \
            : (k2 ? launch_bwd_wide<T, DD, 1, 2>(a, s) : launch_bwd_wide<T, DD, 1, 1>(a, s))
  if (c.dtype == HF_F32) {
    if (c.head_dim == 128) HF_BWD_WIDE(float, 128);
    HF_BWD_WIDE(float, 64);
  }
  if (c.head_dim == 128) HF_BWD_WIDE(bf16_t, 128);
  HF_BWD_WIDE(bf16_t, 64);
#undef HF_BWD_WIDE
}

}  // namespace hf
