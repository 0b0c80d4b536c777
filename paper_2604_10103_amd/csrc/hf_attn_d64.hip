// Block-sparse window attention (Eq. 5) with the history term (Eq. 3, 6) on bf16 MFMA: bf16 storage, head_dim 64.
//
// The layout of the head_dim 128 kernel (hf_attn_mfma.hip): a wavefront owns 32 query rows, tiles of 32 keys, both products
// transposed so that every softmax statistic is private to a lane, K and V tiles global -> LDS directly, V^T fragments by
// transposing reads, three K slots and two V slots, one barrier per tile behind the S^T products.  What differs:
//
//  * Probabilities keep their fp32 bits.  A float is the sum of three bf16 values (8 + 8 + 8 bits of its 24), so
//    P V = hi V + mid V + lo V with three bf16 products per tile instead of one, each exact, all summed in fp32: the
//    arithmetic of an fp32 product of P with bf16 values, at 3/16 of its matrix time.  S = Q K^T needs no split: bf16
//    operands, fp32 sums, scaled in fp32.
//  * O^T takes 32 registers and Q^T 16, so four wavefronts fit on a SIMD and hide each other's chains.
//  * Two groups of two wavefronts share a workgroup's 64 rows, group g the tiles g, g + 2, ... of the list; their partial
//    (m, l, O) meet in LDS at the end and each group finishes half of the features.  A workgroup then has a wavefront on
//    every SIMD: with two wavefronts per workgroup the SIMDs of a compute unit fill unevenly and the last workgroups run
//    twice as long.  (Cases below with one / two / four groups: 37.9 / 28.7 / 28.0 us at 4 heads x 1050 rows, 121 / 110 / 115
//    at 16 x 4200, 178 / 166 / 174 at 24 x 4680, 432 / 413 / 437 at 40 x 6000: two are never far from the best.)
//
// Bound by the vector instructions' issue: half the features per score of head_dim 128, the same softmax per score, plus the
// split.  Per wavefront and tile 16 MFMAs (512 cycles of matrix pipe, ~13 each of the issue port) next to ~530 cycles of vector
// issue (an exponential 8 cycles, three-operand and conversion instructions 4, plain additions and products 2).
// 832x480 with 24 heads of 64 (4680 x 9360, k = 37 of 147 blocks of 64; selection included): 0.66 ms with both products on the
// fp32 matrix instruction, 0.165 ms with this kernel; of those, 12 us are the tiles' transfers, 18 us the selection.
#include <type_traits>

#include "hf_f32_mfma.h"

namespace hf {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

constexpr int D = 64;
constexpr int TK = 32;            // keys per tile
constexpr int ROWB = 2 * D;       // bytes of a token; its eight 16-byte units are permuted in LDS
constexpr int TILE = TK * ROWB;   // 4 KB
constexpr int KS = 2;             // groups of two wavefronts that share a workgroup's rows
constexpr int GB = 5 * TILE;      // a group's tiles: three of K, two of V
constexpr int OSTR = ROWB + 16;   // bytes per query row of the staged output
constexpr float kGrow = 8.0f;     // log2 units: rescale only when a row's maximum grew by more than 2^8

// 16-byte unit u of token row r sits at u ^ swizzle(r).  K: a fragment read takes one unit of 32 rows, 16 lanes at a time;
// two rows share the 64 banks' period, so eight pairs have to fall on eight units whichever row bit separates the halves.
// V: a transposing read takes four units of four rows: rows 0/1 against 2/3 in opposite halves of the row.
__device__ __forceinline__ int k_swizzle(int r) { return ((r >> 1) & 1) | (((r >> 2) ^ (r >> 3)) & 1) << 1 | (((r >> 3) ^ (r >> 4)) & 1) << 2; }
__device__ __forceinline__ int v_swizzle(int r) { return ((r >> 1) & 1) << 2 | ((r >> 2) & 3); }

__device__ __forceinline__ float max3f(float a, float b, float c) {   // (scores are finite or -inf: no NaN quieting)
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}
__device__ __forceinline__ float both_halves_sum(float x) {
  const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
}

__global__ __launch_bounds__(128 * KS, 4) void attn_d64_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V, const int32_t* __restrict__ idx,
    int k, int n_q, int n_kv, int kv_stride, int bq, int bkv, int t_m, int t_n, int chunks, int per_xcd, int total,
    float c_scale, WideHist hist, bf16_t* __restrict__ O) {
  __shared__ __attribute__((aligned(16))) char smem[KS * GB];
  // one contiguous run of (head, query block, 64-row chunk) per XCD: its L2 then holds the keys of few heads
  const int item = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per_xcd || item >= total) return;
  const int bh = item / (t_m * chunks), in_head = item - bh * t_m * chunks;
  const int qb = in_head / chunks, row0 = qb * bq + 64 * (in_head - qb * chunks);
  const int q_end = min(n_q, (qb + 1) * bq);
  if (row0 >= q_end) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = wave & 1, grp = wave >> 1;
  int l32 = lane & 31, h = lane >> 5;
  char* const sK = smem + grp * GB;
  char* const sV = sK + 3 * TILE;
  const int32_t* row_idx = idx ? idx + ((size_t)bh * t_m + qb) * k : nullptr;
  const int nsel = idx ? k : t_n;
  const int subs = bkv / TK;
  const int ntiles = (nsel * subs + KS - 1) / KS;   // every group the same number: the barriers are the workgroup's

  // this lane's query row as B-operand fragments (features 16 s + 8 h .. + 8); rows past the block's end read clamped
  // addresses and are never stored
  auto query_row = [&]() { return row0 + 32 * wr + l32; };
  auto query_at = [&]() { return (size_t)bh * n_q + min(query_row(), n_q - 1); };
  bf16x8 qf[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) qf[s] = *reinterpret_cast<const bf16x8*>(Q + query_at() * D + 16 * s + 8 * h);

  f32x16 o[2];
#pragma unroll
  for (int dt = 0; dt < 2; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[dt][r] = 0.0f;
  float m_ref = -INFINITY, l_run = 0.0f;

  // tiles of the group's part of the list, 64 at a time, lane l holding tile t0 + l: first key | real keys << 24.  Tiles past
  // the end, empty parts of short blocks and indices out of range hold no real key: they start at the head's end, where
  // rows read as zeros (a real row of weight zero would pass a NaN or an infinity on).
  int d_tile = 0, tq = 0;
  auto refill = [&](int t0) {
    const int t = grp + KS * (t0 + lane);
    const int sel = t / subs, sub = t - sel * subs;
    const int jb = row_idx ? row_idx[min(sel, nsel - 1)] : min(sel, nsel - 1);
    const bool ok = sel < nsel && (unsigned)jb < (unsigned)t_n;
    const int st = jb * bkv + TK * sub, real = ok ? min(TK, n_kv - st) : 0;
    d_tile = real > 0 ? (st | (real << 24)) : n_kv;
  };
  refill(0);
  auto next_tile = [&](int& start, int& valid) {
    if ((tq & 63) == 0 && tq > 0) refill(tq);  // uniform
    const int d = __builtin_amdgcn_readlane(d_tile, tq & 63);
    start = d & 0xffffff;
    valid = d >> 24;
    ++tq;
  };

  // a tile is four pieces of 1 KB (eight token rows each), two per wavefront; the tile's first key moves into the descriptor,
  // rows past the head's end arrive as zeros
  const uint64_t kbase = reinterpret_cast<uint64_t>(K + (size_t)bh * kv_stride * D);
  const uint64_t vbase = reinterpret_cast<uint64_t>(V + (size_t)bh * kv_stride * D);
  const int head_bytes = n_kv * ROWB;
  const uint32_t sK_lds = (uint32_t)(uintptr_t)sK, sV_lds = (uint32_t)(uintptr_t)sV;
  int k_off[2], v_off[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int r = 8 * (wr + 2 * j) + (lane >> 3), u = lane & 7;
    k_off[j] = r * ROWB + ((u ^ k_swizzle(r)) * 16);
    v_off[j] = r * ROWB + ((u ^ v_swizzle(r)) * 16);
  }
  auto fetch = [&](uint64_t head, uint32_t slot, int start_v, const int (&off)[2]) {
    const int start = __builtin_amdgcn_readfirstlane(start_v);
    const int skip = start * ROWB, left = head_bytes - skip;
    const uint64_t base = head + (uint64_t)(uint32_t)(left > 0 ? skip : 0);
    const i32x4 desc = {(int)(uint32_t)base, (int)(uint32_t)(base >> 32), left > 0 ? left : 0, 0x00020000};
#pragma unroll
    for (int j = 0; j < 2; ++j)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                   :: "s"(slot + (uint32_t)(1024 * (wr + 2 * j))), "v"(off[j]), "s"(desc) : "memory", "m0");
  };

  // LDS read addresses: K unit 2 s + h of row l32; V (feature 32 dt + l32, keys 16 t2 + 8 x + 4 h .. + 4) by transposing reads:
  // a 16-lane group fetches four key rows x 16 features, lane j the chunk (key j / 4, features 4 (j % 4)) of 8 bytes
  uint32_t k_addr[4], v_addr[2][2];
#pragma unroll
  for (int s = 0; s < 4; ++s) k_addr[s] = l32 * ROWB + 16 * ((2 * s + h) ^ k_swizzle(l32));
  const int j16 = lane & 15, grp16 = lane >> 4, key_l = 4 * h + (j16 >> 2);
#pragma unroll
  for (int dt = 0; dt < 2; ++dt)
#pragma unroll
    for (int x = 0; x < 2; ++x)
      v_addr[dt][x] = (8 * x + key_l) * ROWB + 8 * (j16 & 1) +
                      16 * ((4 * dt + 2 * (grp16 & 1) + ((j16 & 3) >> 1)) ^ v_swizzle(8 * x + key_l));   // + 16 rows for t2 = 1

  int start_a, start_b, start_c, va, vb, vc, vd;   // first keys of tiles t + 1 .. t + 3, real keys of tiles t .. t + 3
  {
    int st0;
    next_tile(st0, va);
    fetch(kbase, sK_lds, st0, k_off);
    fetch(vbase, sV_lds, st0, v_off);
    next_tile(start_a, vb);
    fetch(kbase, sK_lds + TILE, start_a, k_off);
    next_tile(start_b, vc);
    fetch(kbase, sK_lds + 2 * TILE, start_b, k_off);
    next_tile(start_c, vd);
  }
  asm volatile("s_waitcnt vmcnt(4)" ::: "memory");   // K and V of tile 0 (K of tiles 1, 2 may fly)
  __syncthreads();
  bf16x8 kf[4];   // K fragments of the tile whose scores come next
#pragma unroll
  for (int s = 0; s < 4; ++s) kf[s] = *reinterpret_cast<const bf16x8*>(sK + k_addr[s]);

  // the pairs (-1, 0) and (0, -1), kept from the compiler: as an inline constant the first is taken for an fp32 -1 by the
  // instruction, which has its bits in the other half
  uint32_t minus_lo_bits, minus_hi_bits;
  asm("s_mov_b32 %0, 0xbf80" : "=s"(minus_lo_bits));
  asm("s_mov_b32 %0, 0xbf800000" : "=s"(minus_hi_bits));
  const bf16x2 minus_lo = __builtin_bit_cast(bf16x2, minus_lo_bits), minus_hi = __builtin_bit_cast(bf16x2, minus_hi_bits);
  // One tile (kslot = t mod 3, par = t mod 2).  Behind the barrier every wavefront is done with K slot kslot and with V slot
  // par ^ 1, so V of tile t + 1 and K of tile t + 3 are requested into them.
  auto tile_step = [&](const int kslot, const int par) {
    f32x16 sacc;
#pragma unroll
    for (int r = 0; r < 16; ++r) sacc[r] = 0.0f;
#pragma unroll
    for (int s = 0; s < 4; ++s) sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s], qf[s], sacc, 0, 0, 0);
    asm volatile("s_waitcnt vmcnt(2)" ::: "memory");   // K of tile t + 1 and V of tile t have landed; K of tile t + 2 may fly
    __syncthreads();
    fetch(vbase, sV_lds + (par ^ 1) * TILE, start_a, v_off);
    fetch(kbase, sK_lds + kslot * TILE, start_c, k_off);
    start_a = start_b;
    start_b = start_c;
    int vnew;
    next_tile(start_c, vnew);
#pragma unroll
    for (int s = 0; s < 4; ++s) kf[s] = *reinterpret_cast<const bf16x8*>(sK + k_addr[s] + ((kslot + 1) % 3) * TILE);

    if (va < TK) {  // keys that do not exist never contribute
      const int mine = va - 4 * h;
#pragma unroll
      for (int r = 0; r < 16; ++r) sacc[r] = 8 * (r >> 2) + (r & 3) < mine ? sacc[r] : -INFINITY;
    }
    float mx;
    {
      const float m0 = max3f(sacc[0], sacc[1], sacc[2]), m1 = max3f(sacc[3], sacc[4], sacc[5]);
      const float m2 = max3f(sacc[6], sacc[7], sacc[8]), m3 = max3f(sacc[9], sacc[10], sacc[11]);
      const float m4 = max3f(sacc[12], sacc[13], sacc[14]), m5 = max3f(m0, m1, m2);
      mx = max3f(max3f(m3, m4, sacc[15]), m5, m5);
      const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
      mx = max3f(__uint_as_float(sw[0]), __uint_as_float(sw[1]), __uint_as_float(sw[1])) * c_scale;  // both lanes of a query agree
    }
    if (__any(mx > m_ref + kGrow)) {   // (any reference is exact in floating point)
      const float m_new = fmaxf(m_ref, mx);
      const float alpha = __builtin_amdgcn_exp2f(m_ref - (m_new == -INFINITY ? 0.0f : m_new));
      m_ref = m_new;
      l_run *= alpha;
#pragma unroll
      for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
    }
    const float m_use = m_ref == -INFINITY ? 0.0f : m_ref;   // nothing seen yet: keep the exponents finite
    float psum = 0.0f;
#pragma unroll
    for (int t2 = 0; t2 < 2; ++t2) {
      bf16x8 pf[3];
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        float p0 = __builtin_amdgcn_exp2f(fmaf(sacc[8 * t2 + e], c_scale, -m_use));
        float p1 = __builtin_amdgcn_exp2f(fmaf(sacc[8 * t2 + e + 1], c_scale, -m_use));
        psum += p0;
        psum += p1;
        asm volatile("" : "+v"(psum));   // now: the split overwrites p
        // p = hi + mid + lo: each remainder is exact (a dot product with (-1, 0) or (0, -1) subtracts the rounded value)
#pragma unroll
        for (int u = 0; u < 3; ++u) {
          const bf16x2 w = {static_cast<__bf16>(p0), static_cast<__bf16>(p1)};
          pf[u][e] = w[0];
          pf[u][e + 1] = w[1];
          if (u < 2) {
            p0 = __builtin_amdgcn_fdot2_f32_bf16(w, minus_lo, p0, false);
            p1 = __builtin_amdgcn_fdot2_f32_bf16(w, minus_hi, p1, false);
          }
        }
      }
#pragma unroll
      for (int dt = 0; dt < 2; ++dt) {
        const char* p = sV + v_addr[dt][0] + par * TILE + 16 * ROWB * t2;
        const char* q = sV + v_addr[dt][1] + par * TILE + 16 * ROWB * t2;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(q));
        const s16x8 both = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        const bf16x8 vf = __builtin_bit_cast(bf16x8, both);
#pragma unroll
        for (int u = 2; u >= 0; --u) o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[u], o[dt], 0, 0, 0);
      }
    }
    l_run += psum;
    va = vb;
    vb = vc;
    vc = vd;
    vd = vnew;
  };
  for (int t = 0; t < ntiles; t += 6) {   // every (t mod 3, t mod 2) once: slot offsets are immediates
    tile_step(0, 0);
    if (t + 1 >= ntiles) break;
    tile_step(1, 1);
    if (t + 2 >= ntiles) break;
    tile_step(2, 0);
    if (t + 3 >= ntiles) break;
    tile_step(0, 1);
    if (t + 4 >= ntiles) break;
    tile_step(1, 0);
    if (t + 5 >= ntiles) break;
    tile_step(2, 1);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // nothing may land in LDS after the tiles' space is reused
  __syncthreads();
  // (the lane's place opaque from here on: what is formed of it is not kept, or spilled, over the loop)
  int place = lane;
  asm volatile("" : "+v"(place));
  l32 = place & 31;
  h = place >> 5;
  const int q_row = query_row();
  const size_t q_at = query_at();
  float l_tot = both_halves_sum(l_run);

  // ---- the groups' parts of a row meet: [wavefront][feature block][quad][lane] in each group's tile space, then the row
  // statistics; each group finishes one 32-feature block
  f32x4* part = reinterpret_cast<f32x4*>(sK) + wr * 512 + place;
#pragma unroll
  for (int dt = 0; dt < 2; ++dt)
#pragma unroll
    for (int rq = 0; rq < 4; ++rq)
      part[(4 * dt + rq) * 64] = f32x4{o[dt][4 * rq], o[dt][4 * rq + 1], o[dt][4 * rq + 2], o[dt][4 * rq + 3]};
  if (h == 0) {
    float* stat = reinterpret_cast<float*>(sK + 4 * TILE) + 2 * (32 * wr + l32);
    stat[0] = m_ref;
    stat[1] = l_tot;
  }
  __syncthreads();
  float mu[KS], lu[KS];
  m_ref = -INFINITY;
#pragma unroll
  for (int u = 0; u < KS; ++u) {
    const float* q = reinterpret_cast<const float*>(smem + u * GB + 4 * TILE) + 2 * (32 * wr + l32);
    mu[u] = q[0];
    lu[u] = q[1];
    m_ref = fmaxf(m_ref, mu[u]);
  }
  const float m_use = m_ref == -INFINITY ? 0.0f : m_ref;
  l_tot = 0.0f;
  f32x16 os = {};
#pragma unroll
  for (int u = 0; u < KS; ++u) {
    const float w = __builtin_amdgcn_exp2f(mu[u] - m_use);
    l_tot = fmaf(lu[u], w, l_tot);
    const f32x4* q = reinterpret_cast<const f32x4*>(smem + u * GB) + wr * 512 + 4 * grp * 64 + place;
#pragma unroll
    for (int rq = 0; rq < 4; ++rq) {
      const f32x4 x = q[rq * 64];
#pragma unroll
      for (int e = 0; e < 4; ++e) os[4 * rq + e] = fmaf(x[e], w, os[4 * rq + e]);
    }
  }
  // ---- a selected infinity: the small terms of the split made NaN of it (0 inf, inf - inf).  What is not finite is summed again,
  // p v on the fp32 instruction, operands straight from memory (K pieces of a row, V a key's 32 features); where the weights
  // themselves are not finite NaN is right.  Finite inputs never get here.  One infinite value or NaN that every query block selects:
  // 24 heads x 4680 x 9360, k = 37 of 147 blocks of 64, 148 -> 500 us (key after key it
  // took 11360).
  bool bad = false;
#pragma unroll
  for (int r = 0; r < 16; ++r) bad |= !(fabsf(os[r]) < INFINITY);
  if (__any(bad && l_tot < INFINITY)) {
    f32x16 again = {};
    const bf16_t* qp = Q + q_at * D + 8 * h;
    bf16x8 qa[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) qa[s] = *reinterpret_cast<const bf16x8*>(qp + 16 * s);
    const size_t head = (size_t)bh * kv_stride * D;
    const int k_at = l32 * ROWB + 16 * h, v_at = 4 * h * ROWB + 2 * (32 * grp + l32);
#pragma unroll 1
    for (int t = 0; t < nsel * subs; ++t) {
      const int sel = t / subs, jb = __builtin_amdgcn_readfirstlane(row_idx ? row_idx[sel] : sel);
      if ((unsigned)jb >= (unsigned)t_n) continue;
      const int first = jb * bkv + TK * (t - sel * subs), cnt = min(TK, n_kv - first);
      if (cnt <= 0) continue;
      const __amdgpu_buffer_rsrc_t kr = tile_rows<bf16_t, D>(K + head, first, cnt), vr = tile_rows<bf16_t, D>(V + head, first, cnt);
      f32x16 sc = {};
#pragma unroll
      for (int s = 0; s < 4; ++s)
        sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(kr, k_at + 32 * s, 0, 0)),
                                                     qa[s], sc, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 16; ++r)
        sc[r] = 8 * (r >> 2) + (r & 3) < cnt - 4 * h ? __builtin_amdgcn_exp2f(fmaf(sc[r], c_scale, -m_use)) : 0.0f;
#pragma unroll
      for (int rq = 0; rq < 4; ++rq)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t v = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(vr, v_at + (8 * rq + e) * ROWB, 0, 0);
          again = mfma_f32_wide(__uint_as_float(v << 16), sc[4 * rq + e], again);
        }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) os[r] = fabsf(os[r]) < INFINITY ? os[r] : again[r];
  }
  float w = l_tot > 0.0f ? 1.0f / l_tot : 0.0f;   // a row without a single real key: O_local = 0
  if (hist.L) {
    // ---- O += R(phi(q)) L / (z_scale phi(q).z + eps) (Eq. 3, 6) on the fp32 matrix instruction, whose results lie as those
    // of the bf16 one: O_local is scaled by the denominator, the products add the numerator, one division at the end
    const size_t trow = (size_t)min(q_row, n_q - 1) * (D / 2);
    // the lane's features 16 s + 8 h .. + 8, s < 4, in one round trip and in their storage type, L's rows of half of them at a
    // time (as floats, or with an address per row of L, they do not fit the registers: fifteen went to scratch, which cost launches
    // without a state too, 10 heads x 640 rows x 128 keys 6.48 -> 6.13 us)
    const float* z = hist.z + (size_t)bh * D + 8 * h;
    const bf16_t* qp = static_cast<const bf16_t*>(hist.q_hist) + q_at * D + 8 * h;
    bf16x8 qh[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) qh[s] = *reinterpret_cast<const bf16x8*>(qp + 16 * s);
    const __amdgpu_buffer_rsrc_t L = tile_rows<float, D>(hist.L + (size_t)bh * D * D, 0, D);
    const int l_at = (8 * h * D + 32 * grp + l32) * 4;
    float a[16];
    auto rows_of = [&](int s0) {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        a[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(L, l_at, (16 * (s0 + (i >> 3)) + (i & 7)) * D * 4, 0));
    };
    rows_of(0);
    float den = 0.0f;
    auto readout = [&](auto relu) {
      auto piece = [&](int s, int e0) {
        f32x4 x;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = phi_apply(static_cast<float>(qh[s][e0 + e]), relu.value ? HF_PHI_RELU : HF_PHI_ELU1);
        return x;
      };
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const f32x4 zz = *reinterpret_cast<const f32x4*>(z + 16 * (i >> 1) + 4 * (i & 1)), x = piece(i >> 1, 4 * (i & 1));
#pragma unroll
        for (int e = 0; e < 4; ++e) den = fmaf(x[e], zz[e], den);
      }
      den = hist.z_scale * both_halves_sum(den) + hist.eps;
      w *= den;
#pragma unroll
      for (int r = 0; r < 16; ++r) os[r] *= w;
#pragma unroll
      for (int s = 0; s < 4; ++s) asm volatile("" : "+v"(qh[s]));   // (opaque: what the denominator made of them is not kept)
#pragma unroll
      for (int s0 = 0; s0 < 4; s0 += 2) {
        f32x2 cs[4], sn[4];
        if (hist.cosq) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const size_t at = trow + 4 * h + 8 * (s0 + (i >> 1)) + 2 * (i & 1);
            cs[i] = *reinterpret_cast<const f32x2*>(hist.cosq + at);
            sn[i] = *reinterpret_cast<const f32x2*>(hist.sinq + at);
          }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          f32x4 x = piece(s0 + (i >> 1), 4 * (i & 1));
          if (hist.cosq) x = rotate4(x, cs[i][0], sn[i][0], cs[i][1], sn[i][1]);
#pragma unroll
          for (int e = 0; e < 4; ++e) os = mfma_f32_wide(a[4 * i + e], x[e], os);
        }
        if (s0 == 0) rows_of(2);
      }
    };
    if (hist.phi_kind == HF_PHI_RELU) readout(std::true_type{}); else readout(std::false_type{});   // uniform
    w = 1.0f / den;
  }
  // ---- rows through LDS, stored coalesced
  __syncthreads();   // every part has been read
#pragma unroll
  for (int rq = 0; rq < 4; ++rq)
    store4<bf16_t>(reinterpret_cast<bf16_t*>(smem + (32 * wr + l32) * OSTR) + 32 * grp + 8 * rq + 4 * h,
                   f32x4{os[4 * rq], os[4 * rq + 1], os[4 * rq + 2], os[4 * rq + 3]} * w);
  __syncthreads();
  for (int e = 64 * wave + place; e < 64 * 8; e += 128 * KS) {
    const int row = e >> 3, u = e & 7;
    if (row0 + row < q_end)
      *reinterpret_cast<uint4*>(O + ((size_t)bh * n_q + row0 + row) * D + 8 * u) =
          *reinterpret_cast<const uint4*>(smem + row * OSTR + 16 * u);
  }
}

}  // namespace

// the descriptors hold the first key in 24 bits
bool attn_d64_supported(const hf_config& c, int n_kv) {
  return c.dtype == HF_BF16 && c.head_dim == D && c.block_q % 64 == 0 && c.block_kv % TK == 0 && n_kv < (1 << 23);
}

int launch_attn_d64(const hf_config& c, const void* Q, int n_q, const void* K, const void* V, int n_kv, const int32_t* idx,
                    int k, void* O, const WideHist& hist, hipStream_t s) {
  const int t_m = (n_q + c.block_q - 1) / c.block_q, t_n = (n_kv + c.block_kv - 1) / c.block_kv;
  const int chunks = c.block_q / 64;
  const long long total = (long long)c.batch * c.heads * t_m * chunks;
  if (total > (1ll << 30)) { set_error("too many query blocks"); return HF_ERR_SHAPE; }
  const int per_xcd = (int)((total + 7) / 8);
  const float scale = c.softmax_scale > 0.0f ? c.softmax_scale : 1.0f / sqrtf((float)D);
  hipLaunchKernelGGL(attn_d64_kernel, dim3(8 * per_xcd), dim3(128 * KS), 0, s, static_cast<const bf16_t*>(Q),
                     static_cast<const bf16_t*>(K), static_cast<const bf16_t*>(V), idx, k, n_q, n_kv, kv_stride_of(c, n_kv),
                     c.block_q, c.block_kv, t_m, t_n, chunks, per_xcd, (int)total, scale * 1.4426950408889634f, hist,
                     static_cast<bf16_t*>(O));
  return check_launch("hf_hybrid_attn_fwd(attention)");
}

}  // namespace hf
