// Block-sparse window attention (Eq. 5) for fp32 storage on the bf16 matrix instruction, and the history term (Eq. 3, 6): block_q
// a multiple of 64, block_kv of 32.
//
// An fp32 value is the sum of three bf16 values, x = hi + mid + lo, each the rest so far rounded to nearest: |mid| <= 2^-8 and
// |lo| <= 2^-17 of x's leading bit, the remainders exact.  A product of two of them is six bf16 products, each exact, summed in
// fp32 by the matrix cores:
//   x y = hi hi' + (hi mid' + mid hi') + (hi lo' + mid mid' + lo hi')
// What is left out, mid lo' + lo mid' + lo lo', is at most 2^-24 of the product (one rounding to fp32) and of either sign.  (Parts
// below 2^-133 vanish: a score is off by 2^-134 of the other operand, which counts next to one above 2^100 alone; outputs so small
// are formed again behind the loop.)
// The bf16 instruction has sixteen times the rate of the fp32 one, so six products take 6/16 of its matrix time, and a sum is
// rounded once per sixteen terms instead of once per two.  A tile's P V is summed for itself and added to the output once.
// Against 64 bits, with both products on the fp32 instruction / here (32 to 4096 keys): Gaussian inputs of standard deviation 0.5
// 1.3e-7..5.9e-7 / 1.0e-7..2.1e-7, 1 2.5e-7..7.2e-7 / 1.8e-7..3.7e-7, 2 4.3e-7..1.7e-6 / 3.1e-7..1.2e-6; low fifteen bits all
// set, both signs 1.2e-7..6.0e-7 / 0.8e-7..1.9e-7, one sign 0.75e-7..2.7e-7 / 0.76e-7..1.2e-7.  Parts cut off instead of rounded leave out
// up to 2^-21, always of the product's sign: with such inputs up to 1.2 times the error of the fp32 instruction, for 16 us less
// of 468 (832x480).  Eight products (2^-30 left out) take 545.
//
// Layout as in the bf16 kernels (hf_attn_mfma.hip): a wavefront owns 32 query rows and walks tiles of 32 keys, both products are
// formed transposed (S^T = K Q^T, O^T += V^T P^T), a lane's sixteen scores belong to one query, and the exponentials split into
// their three parts are the B operand of the second product.  What differs is how a tile gets to LDS: the workgroup's two
// wavefronts of rows load it as fp32 (in registers one phase before its use), split it once for both and store three
// bf16 planes.  A workgroup has KG groups of two wavefronts with every KG-th tile of the list each; the groups' (m, l, O) meet
// in LDS behind the loop and every group finishes DT / KG feature blocks.  Of the three planes of Q two stay in registers, the
// third (one product of six) in LDS.
//
// 832x480 in fp32 (12 heads of 128, 4680 x 9360, k = 37 of 147 blocks of 64; selection included): 613 us on the fp32 instruction,
// 468 here.  Splitting next to the matrix instructions instead of behind them, transposing reads for V, and remainders by dot
// products with (-1, 0) instead of subtractions (they run on the matrix pipe) gained nothing.
#include <type_traits>

#include "hf_f32_mfma.h"

namespace hf {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr int TK = 32;            // keys per tile
constexpr int RG = 2;             // wavefronts along the rows
constexpr float kGrow = 8.0f;     // log2 units: rescale only when a row's maximum grew by more than 2^8

// Keys: 16-byte unit u of row r sits at u ^ swizzle(r), and fragment reads (one unit of 32 rows) are free of bank conflicts; what
// is written at a time is whole rows.
template <int D> __device__ __forceinline__ int k_swizzle(int r) {
  if (D == 128) return r & 15;
  return ((r >> 1) & 1) | (((r >> 2) ^ (r >> 3)) & 1) << 1 | (((r >> 3) ^ (r >> 4)) & 1) << 2;
}
// Values lie transposed, 32 keys of a feature in 64 bytes: unit 2 t2 + h holds the keys 16 t2 + 8 x + 4 h + 0..3, x = 0, 1, which is
// what a lane of the second product's A operand takes.  Features are permuted so that eight lanes' writes (features D / 32 apart)
// and sixteen lanes' reads (features one apart, any one of their bits 2 to 4 alike) fall on different banks.
__device__ __forceinline__ int v_place(int f, int unit) {
  return 64 * (f ^ (((f >> 1) ^ (f >> 2)) & 1)) + 16 * (unit ^ ((((f >> 2) ^ (f >> 3)) & 1) | (((f >> 3) ^ (f >> 4)) & 1) << 1));
}

__device__ __forceinline__ float both_halves_sum(float x) {
  const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
}

// Eight values split together.  (The last remainder has at most eight significant bits: its upper half is all of it.)
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
struct Split {
  u32x4 part[3];
  float x[8];
  __device__ __forceinline__ bf16x8 operator[](int u) const { return __builtin_bit_cast(bf16x8, part[u]); }
  __device__ __forceinline__ void all() {
#pragma unroll
    for (int u = 0; u < 3; ++u) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (u == 2) {
          part[u][e] = __builtin_amdgcn_perm(__float_as_uint(x[2 * e + 1]), __float_as_uint(x[2 * e]), 0x07060302u);
          continue;
        }
        part[u][e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x[2 * e], x[2 * e + 1]}, bf16x2));
        x[2 * e] -= __uint_as_float(part[u][e] << 16);
        x[2 * e + 1] -= __uint_as_float(part[u][e] & 0xffff0000u);
      }
    }
  }
};
__device__ __forceinline__ f32x16 mfma_bf16(const bf16x8& a, const bf16x8& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
// the six products of operands in three parts each, smallest first: factors of product i
__device__ __forceinline__ constexpr int prod_a(int i) { return i == 0 ? 2 : (i == 2 || i == 3) ? 1 : 0; }
__device__ __forceinline__ constexpr int prod_b(int i) { return i == 1 ? 2 : (i == 2 || i == 4) ? 1 : 0; }

template <int D, int KG>
struct SplitShape {
  static constexpr int WAVES = D == 128 ? 2 : (KG == 1 ? 3 : 2);   // wavefronts per SIMD that the registers allow
  static constexpr int ROWB = 2 * D;                        // bytes of a token in a plane
  static constexpr int PLANE = TK * ROWB;
  static constexpr int QL = 32 * RG * ROWB;                 // third plane of the queries
  static constexpr int BUDGET = 40960 / WAVES * RG * KG;    // LDS of a workgroup if that many wavefronts are to fit
  static constexpr bool TWO = QL + 2 * KG * 3 * PLANE <= BUDGET;   // keys and values have a place each
  static constexpr int GBUF = (TWO ? 6 : 3) * PLANE;
  static constexpr int DT = D / 32, ND = DT / KG;
  static constexpr int STAGE = 32 * RG * (D + 4) * 4;       // output rows
  static constexpr int MEET = KG > 1 ? 32 * RG * KG * 8 + KG * (DT - ND) * RG * 4096 : 0;
  static constexpr int TILES = QL + KG * GBUF;
  static constexpr int LDS = TILES > STAGE ? (TILES > MEET ? TILES : MEET) : (STAGE > MEET ? STAGE : MEET);
};

template <int D, int KG>
__global__ __launch_bounds__(64 * RG * KG, (SplitShape<D, KG>::WAVES)) void attn_split_kernel(
    const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V, const int32_t* __restrict__ idx,
    int k, int n_q, int n_kv, int kv_stride, int bq, int bkv, int t_m, int t_n, int chunks, int per_xcd, int total,
    float scale_log2e, WideHist hist, float* __restrict__ O) {
  using Sh = SplitShape<D, KG>;
  constexpr int NT = 64 * RG * KG, ROWB = Sh::ROWB, PLANE = Sh::PLANE, DT = Sh::DT, ND = Sh::ND, S = D / 16;
  constexpr int NP = TK * D / (64 * RG) / 8;            // eights of elements that a lane brings of a tile
  constexpr int OST = D + 4;                            // floats per row of the staged output
  __shared__ __attribute__((aligned(16))) char smem[Sh::LDS];
  // one contiguous run of (head, query block, chunk of rows) per XCD: its L2 then holds the keys of few heads
  const int item = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= per_xcd || item >= total) return;
  const int bh = item / (t_m * chunks), in_head = item - bh * t_m * chunks;
  const int qb = in_head / chunks, row0 = qb * bq + 32 * RG * (in_head - qb * chunks);
  const int q_end = min(n_q, (qb + 1) * bq);
  if (row0 >= q_end) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = wave % RG, grp = wave / RG;
  int l32 = lane & 31, h = lane >> 5;
  char* const sK = smem + Sh::QL + grp * Sh::GBUF;
  char* const sV = sK + (Sh::TWO ? 3 * PLANE : 0);
  const float* Kh = K + (size_t)bh * kv_stride * D;     // heads of a cache buffer are kv_stride tokens apart
  const float* Vh = V + (size_t)bh * kv_stride * D;
  const int32_t* row_idx = idx ? idx + ((size_t)bh * t_m + qb) * k : nullptr;
  const int nsel = idx ? k : t_n;
  const int subs = bkv / TK;
  const int ntiles = (nsel * subs + KG - 1) / KG;       // every group the same number: the barriers are the workgroup's
  // rows past the block's end: clamped addresses, never written
  auto query_row = [&]() { return row0 + 32 * wr + l32; };
  auto query_at = [&]() { return ((size_t)bh * n_q + min(query_row(), n_q - 1)) * D; };

  // tiles of the group's part of the list, 64 at a time, lane l holding tile t0 + l: first key | real keys << 24; none past the
  // end, for empty parts of short blocks and for indices out of range (rows that do not exist read as zeros)
  int d_tile = 0, tq = 0;
  auto refill = [&](int t0) {
    const int t = grp + KG * (t0 + lane);
    const int sel = t / subs, sub = t - sel * subs;
    const int jb = row_idx ? row_idx[min(sel, nsel - 1)] : min(sel, nsel - 1);
    const bool ok = sel < nsel && (unsigned)jb < (unsigned)t_n;
    const int st = jb * bkv + TK * sub, real = ok ? min(TK, n_kv - st) : 0;
    d_tile = real > 0 ? (st | (real << 24)) : 0;
  };
  refill(0);
  auto next_tile = [&](int& start, int& valid) {
    if ((tq & 63) == 0 && tq > 0) refill(tq);  // uniform
    const int d = __builtin_amdgcn_readlane(d_tile, tq & 63);
    start = d & 0xffffff;
    valid = d >> 24;
    ++tq;
  };

  // ---- a tile's way: fp32 rows into registers, three bf16 planes into LDS.  Keys: a lane eight features of NP rows.  Values: a
  // lane eight keys (a unit) of NP features.
  constexpr int UPR = D / 8, RPP = 64 / UPR;            // units per row of keys, rows that a wavefront loads at a time
  static_assert(NP == D / 32 && NP == TK / RPP / RG, "a wavefront brings half of a tile");
  typedef float vrow __attribute__((ext_vector_type(NP)));
  const int w_row = RPP * wr + lane / UPR, unit = lane % UPR;
  int k_at = (w_row * D + 8 * unit) * 4, v_at = ((16 * wr + 4 * h) * D + NP * l32) * 4;
  // (the swizzle is linear in the row's bits: that of a row a multiple of a power of two further on is the exclusive or of both)
  int k_wr = w_row * ROWB + 16 * (unit ^ k_swizzle<D>(w_row));
  int v_wr[NP];
#pragma unroll
  for (int j = 0; j < NP; ++j) v_wr[j] = v_place(NP * l32 + j, 2 * wr + h);
  Split cv[NP];
  auto load_k = [&](int first, int cnt) {
    const __amdgpu_buffer_rsrc_t rows = tile_rows<float, D>(Kh, first, cnt);
#pragma unroll
    for (int j = 0; j < NP; ++j)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const f32x4 v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rows, k_at + j * RPP * RG * D * 4 + 16 * e, 0, 0));
#pragma unroll
        for (int i = 0; i < 4; ++i) cv[j].x[4 * e + i] = v[i];
      }
  };
  auto load_v = [&](const float* head, int first, int cnt) {
    const __amdgpu_buffer_rsrc_t rows = tile_rows<float, D>(head, first, cnt);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int at = v_at + (8 * (i >> 2) + (i & 3)) * D * 4;
      vrow v;
      if constexpr (NP == 4) v = __builtin_bit_cast(vrow, __builtin_amdgcn_raw_buffer_load_b128(rows, at, 0, 0));
      else v = __builtin_bit_cast(vrow, __builtin_amdgcn_raw_buffer_load_b64(rows, at, 0, 0));
#pragma unroll
      for (int j = 0; j < NP; ++j) cv[j].x[i] = v[j];
    }
  };
  auto write_k = [&]() {
#pragma unroll
    for (int u = 0; u < 3; ++u)
#pragma unroll
      for (int j = 0; j < NP; ++j)
        *reinterpret_cast<u32x4*>(sK + u * PLANE + (k_wr ^ 16 * k_swizzle<D>(RPP * RG * j)) + RPP * RG * j * ROWB) = cv[j].part[u];
  };
  auto write_v = [&]() {
#pragma unroll
    for (int u = 0; u < 3; ++u)
#pragma unroll
      for (int j = 0; j < NP; ++j) *reinterpret_cast<u32x4*>(sV + u * PLANE + v_wr[j]) = cv[j].part[u];
  };
  auto split_tile = [&]() {
#pragma unroll
    for (int j = 0; j < NP; ++j) {
      cv[j].all();
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // LDS read addresses: K unit 2 s + h of row l32; V unit 2 t2 + h of feature 32 dt + l32 (whose places are 2 KB apart)
  int k_rd = l32 * ROWB + 16 * (h ^ k_swizzle<D>(l32));   // ^ 32 s
  int q_rd = k_rd + 32 * wr * ROWB;                       // likewise, of the workgroup's queries
  int v_rd = v_place(l32, h);                             // ^ 32 t2
  auto k_frag = [&](int s, int u) {   // u = 3: third plane of the queries
    const int at = (u < 3 ? k_rd : q_rd) ^ (32 * s);
    return *reinterpret_cast<const bf16x8*>((u < 3 ? sK + u * PLANE : smem) + at);
  };
  auto v_frag = [&](const char* plane, int dt, int t2) {
    return *reinterpret_cast<const bf16x8*>(plane + (v_rd ^ (32 * t2)) + 2048 * dt);
  };

  int start, valid;
  next_tile(start, valid);
  load_k(start, valid);
  // ---- the scaled queries: B operand (features 16 s + 8 h .. + 8 of row l32), the third plane in LDS
  bf16x8 qf[S][2];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const float* qp = Q + query_at() + 16 * s + 8 * h;
    const f32x4 a = *reinterpret_cast<const f32x4*>(qp) * scale_log2e, b = *reinterpret_cast<const f32x4*>(qp + 4) * scale_log2e;
    Split sp;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      sp.x[e] = a[e];
      sp.x[4 + e] = b[e];
    }
    sp.all();
    qf[s][0] = sp[0];
    qf[s][1] = sp[1];
    if (grp == 0) *reinterpret_cast<u32x4*>(smem + (q_rd ^ (32 * s))) = sp.part[2];   // uniform
  }
  f32x16 o[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[dt][r] = 0.0f;
  float m = -INFINITY, l = 0.0f;
  split_tile();
  write_k();
  load_v(Vh, start, valid);

  for (int t = 0; t < ntiles; ++t) {
    asm volatile("" : "+v"(k_rd), "+v"(q_rd), "+v"(v_rd), "+v"(k_wr));   // (opaque: sums stay out of registers)
    __syncthreads();   // the keys of tile t lie in LDS
    // ---- S^T = K Q^T
    f32x16 sc;
#pragma unroll
    for (int r = 0; r < 16; ++r) sc[r] = 0.0f;
    {
      bf16x8 a[3], ql, na[3], nq;
#pragma unroll
      for (int u = 2; u >= 0; --u) a[u] = k_frag(0, u);
      ql = k_frag(0, 3);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s = 0; s < S; ++s) {
#pragma unroll
        for (int i = 0; i < 6; ++i) {
          const int pb = prod_b(i);
          sc = mfma_bf16(a[prod_a(i)], pb == 0 ? qf[s][0] : pb == 1 ? qf[s][1] : ql, sc);
          if (s + 1 < S) {   // a fragment of the next step as soon as one of this step is done with
            if (i == 0) na[2] = k_frag(s + 1, 2);
            if (i == 1) { na[0] = k_frag(s + 1, 0); nq = k_frag(s + 1, 3); }
            if (i == 3) na[1] = k_frag(s + 1, 1);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int u = 0; u < 3; ++u) a[u] = na[u];
        ql = nq;
      }
    }
    if (!Sh::TWO) __syncthreads();   // everybody has read the keys
    const int valid_cur = valid;
    __builtin_amdgcn_sched_barrier(0);

    if (valid_cur < TK) {   // keys that do not exist never contribute
      const int mine = valid_cur - 4 * h;
#pragma unroll
      for (int r = 0; r < 16; ++r) sc[r] = 8 * (r >> 2) + (r & 3) < mine ? sc[r] : -INFINITY;
    }
    float mx = sc[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, sc[r]);
    {
      const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
      mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));   // both lanes of a query agree
    }
    if (__any(mx > m + kGrow)) {   // (any reference is exact in floating point)
      const float m_new = fmaxf(m, mx);
      const float alpha = __builtin_amdgcn_exp2f(m - (m_new == -INFINITY ? 0.0f : m_new));
      m = m_new;
      l *= alpha;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
    }
    const float m_use = m == -INFINITY ? 0.0f : m;   // nothing seen yet: keep the exponents finite
    Split p[2];
    float psum[2];
#pragma unroll
    for (int t2 = 0; t2 < 2; ++t2) {
#pragma unroll
      for (int e = 0; e < 8; ++e) p[t2].x[e] = __builtin_amdgcn_exp2f(sc[8 * t2 + e] - m_use);
      psum[t2] = ((p[t2].x[0] + p[t2].x[1]) + (p[t2].x[2] + p[t2].x[3])) + ((p[t2].x[4] + p[t2].x[5]) + (p[t2].x[6] + p[t2].x[7]));
      __builtin_amdgcn_sched_barrier(0);
      p[t2].all();
      __builtin_amdgcn_sched_barrier(0);
    }
    l += psum[0] + psum[1];
    split_tile();
    write_v();
    next_tile(start, valid);
    load_k(start, valid);
    __builtin_amdgcn_sched_barrier(0);

    __syncthreads();   // the values of tile t lie in LDS
    // ---- O^T += V^T P^T, the tile's sum for itself: one addition per tile at the accumulator's magnitude
    {
      constexpr int U = 2 * DT;   // (feature block, half of the tile)
      bf16x8 a[3], na[3];
#pragma unroll
      for (int u = 2; u >= 0; --u) a[u] = v_frag(sV + u * PLANE, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        f32x16 part;
#pragma unroll
        for (int r = 0; r < 16; ++r) part[r] = 0.0f;
#pragma unroll
        for (int t2 = 0; t2 < 2; ++t2) {
          const int c = 2 * dt + t2;
#pragma unroll
          for (int i = 0; i < 6; ++i) {
            part = mfma_bf16(a[prod_a(i)], p[t2][prod_b(i)], part);
            if (c + 1 < U) {
              if (i == 0) na[2] = v_frag(sV + 2 * PLANE, (c + 1) >> 1, (c + 1) & 1);
              if (i == 1) na[0] = v_frag(sV, (c + 1) >> 1, (c + 1) & 1);
              if (i == 3) na[1] = v_frag(sV + PLANE, (c + 1) >> 1, (c + 1) & 1);
            }
            __builtin_amdgcn_sched_barrier(0);
          }
#pragma unroll
          for (int u = 0; u < 3; ++u) a[u] = na[u];
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] += part[r];
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    split_tile();
    if (!Sh::TWO) __syncthreads();   // everybody has read the values
    write_k();
    load_v(Vh, start, valid);
    __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();
  // (the lane's place opaque from here on: what is formed of it is not kept over the loop)
  int place = lane;
  asm volatile("" : "+v"(place));
  l32 = place & 31;
  h = place >> 5;
  const int row = query_row();
  const size_t q_at = query_at();
  float l_tot = both_halves_sum(l);

  if (KG > 1) {
    // ---- the groups' parts of a row meet: row statistics, then [group][block of another group][wavefront][quad][lane]
    float2* const stat = reinterpret_cast<float2*>(smem);
    f32x4* const parts = reinterpret_cast<f32x4*>(smem + 32 * RG * KG * 8) + lane;
    auto part_at = [&](int u, int dt) {   // where group u keeps block dt
      const int slot = dt - (dt / ND > u ? ND : 0);
      return parts + ((u * (DT - ND) + slot) * RG + wr) * 256;
    };
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
      if (dt / ND != grp) {   // uniform
        f32x4* q = part_at(grp, dt);
#pragma unroll
        for (int rq = 0; rq < 4; ++rq) q[rq * 64] = f32x4{o[dt][4 * rq], o[dt][4 * rq + 1], o[dt][4 * rq + 2], o[dt][4 * rq + 3]};
      }
    if (h == 0) stat[(32 * wr + l32) * KG + grp] = make_float2(m, l_tot);
    __syncthreads();
    const float m_own = m;
    float wu[KG], lu[KG];
#pragma unroll
    for (int u = 0; u < KG; ++u) {
      const float2 st = stat[(32 * wr + l32) * KG + u];
      wu[u] = st.x;
      lu[u] = st.y;
      m = fmaxf(m, st.x);
    }
    const float m_use = m == -INFINITY ? 0.0f : m;
    l_tot = 0.0f;
#pragma unroll
    for (int u = 0; u < KG; ++u) {
      wu[u] = __builtin_amdgcn_exp2f(wu[u] - m_use);
      l_tot = fmaf(lu[u], wu[u], l_tot);
    }
    const float w_own = __builtin_amdgcn_exp2f(m_own - m_use);
    // this group's blocks move to the front (constant indices: accumulators stay in registers)
#pragma unroll
    for (int g = 1; g < KG; ++g)
      if (grp == g) {   // uniform
#pragma unroll
        for (int i = 0; i < ND; ++i) o[i] = o[ND * g + i];
      }
#pragma unroll
    for (int i = 0; i < ND; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[i][r] *= w_own;
#pragma unroll
    for (int u = 0; u < KG; ++u)
      if (u != grp) {   // uniform; group order
#pragma unroll
        for (int i = 0; i < ND; ++i) {
          const f32x4* q = part_at(u, ND * grp + i);
#pragma unroll
          for (int rq = 0; rq < 4; ++rq) {
            const f32x4 x = q[rq * 64];
#pragma unroll
            for (int e = 0; e < 4; ++e) o[i][4 * rq + e] = fmaf(x[e], wu[u], o[i][4 * rq + e]);
          }
        }
      }
    __syncthreads();   // every part has been read
  }
  const int f0 = 32 * ND * grp;   // o[i], i < ND, holds features f0 + 32 i .. + 32 from here on

  // ---- what is not finite: an infinity has no finite remainder (inf - inf), and the small terms of the split multiply it by
  // zero.  And what is below 2^-106: the third part of such a value lies under bf16's smallest (2^-133; an output of 2^-120 was off by
  // 3.5e-5 of itself).  A wavefront with such a row does its rows again on the fp32 instruction, operands straight from memory (K and Q pieces
  // of a row, V a key's 32 features), and takes the rows that need it.  Finite inputs up to bf16's largest value never get here; one
  // infinite value or NaN that every query block selects: 832x480 470 -> 1350 us (620 with fp32
  // products throughout; key after key took 13400).
  {
    float bad = l_tot < INFINITY ? 0.0f : 1.0f;
    const float tiny = l_tot * 0x1p-106f;
#pragma unroll
    for (int i = 0; i < ND; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float a = fabsf(o[i][r]);
        bad = a == 0.0f || (a >= tiny && a < INFINITY) ? bad : 1.0f;
      }
    bad = both_halves_sum(bad);
    if (__any(bad > 0.0f)) {
      f32x16 again[ND];
#pragma unroll
      for (int i = 0; i < ND; ++i) again[i] = {};
      float m2 = -INFINITY, l2 = 0.0f;
      const float* qp = Q + q_at + 4 * h;
      const int k2_at = (l32 * D + 4 * h) * 4, v2_at = (4 * h * D + f0 + l32) * 4;
#pragma unroll 1
      for (int t = 0; t < nsel * subs; ++t) {
        const int sel = t / subs, jb = __builtin_amdgcn_readfirstlane(row_idx ? row_idx[sel] : sel);
        if ((unsigned)jb >= (unsigned)t_n) continue;
        const int first = jb * bkv + TK * (t - sel * subs), cnt = min(TK, n_kv - first);
        if (cnt <= 0) continue;
        const __amdgpu_buffer_rsrc_t kr = tile_rows<float, D>(Kh, first, cnt), vr = tile_rows<float, D>(Vh, first, cnt);
        f32x16 sc = {};
#pragma unroll 1
        for (int i0 = 0; i0 < D / 8; i0 += 4) {
          f32x4 x[4], y[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            y[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(kr, k2_at + 32 * (i0 + i), 0, 0));
            x[i] = *reinterpret_cast<const f32x4*>(qp + 8 * (i0 + i)) * scale_log2e;
          }
#pragma unroll
          for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) sc = mfma_f32_wide(y[i][e], x[i][e], sc);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) sc[r] = 8 * (r >> 2) + (r & 3) < cnt - 4 * h ? sc[r] : -INFINITY;
        float mx = sc[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) mx = fmaxf(mx, sc[r]);
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
        mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
        if (__any(mx > m2 + kGrow)) {
          const float m_new = fmaxf(m2, mx);
          const float alpha = __builtin_amdgcn_exp2f(m2 - (m_new == -INFINITY ? 0.0f : m_new));
          m2 = m_new;
          l2 *= alpha;
#pragma unroll
          for (int i = 0; i < ND; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) again[i][r] *= alpha;
        }
        const float ref = m2 == -INFINITY ? 0.0f : m2;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          sc[r] = __builtin_amdgcn_exp2f(sc[r] - ref);
          l2 += sc[r];   // this lane's keys only; summed at the end
        }
#pragma unroll
        for (int rq = 0; rq < 4; ++rq) {
          float v[4][ND];
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < ND; ++i)
              v[e][i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(vr, v2_at + ((8 * rq + e) * D + 32 * i) * 4, 0, 0));
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < ND; ++i) again[i] = mfma_f32_wide(v[e][i], sc[4 * rq + e], again[i]);
        }
      }
      l2 = both_halves_sum(l2);
      if (bad > 0.0f) {
        m = m2;
        l_tot = l2;
#pragma unroll
        for (int i = 0; i < ND; ++i) o[i] = again[i];
      }
    }
  }
  float w = l_tot > 0.0f ? 1.0f / l_tot : 0.0f;   // a row without a single real key: O_local = 0

  if (hist.lse2) {
    // ---- statistics for the backward pass: log2 of the sum of 2^(scaled logit), and D = dO . O_local from the unrounded
    // output, the groups' features of which are summed as scalars
    const float* gp = static_cast<const float*>(hist.d_out) + q_at + f0 + 4 * h;
    float acc = 0.0f;
#pragma unroll
    for (int i = 0; i < ND; ++i)
#pragma unroll
      for (int rq = 0; rq < 4; ++rq) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(gp + 32 * i + 8 * rq);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = fmaf(o[i][4 * rq + e] * w, x[e], acc);
      }
    acc = both_halves_sum(acc);
    if (KG > 1) {
      float* const sum = reinterpret_cast<float*>(smem) + (32 * wr + l32) * KG;
      if (h == 0) sum[grp] = acc;
      __syncthreads();
      acc = 0.0f;
#pragma unroll
      for (int u = 0; u < KG; ++u) acc += sum[u];
    }
    if (h == 0 && grp == 0 && row < q_end) {
      hist.lse2[(size_t)bh * n_q + row] = l_tot > 0.0f ? m + log2f(l_tot) : INFINITY;   // no real key: P = 0
      hist.dvec[(size_t)bh * n_q + row] = acc;
    }
    return;
  }

  if (hist.L) {
    // ---- O += R(phi(q)) L / (z_scale phi(q).z + eps) (Eq. 3, 6): O_local is scaled by the denominator, the products add the
    // numerator (L's key features in the place of keys, R(phi(q)) in that of the exponentials), one division at the end.  On the
    // fp32 instruction: an infinite entry of the state has no finite remainder, and of a head's products these are D / (k block_kv).
    // A lane takes features 8 i + 4 h .. + 4 of its query and the rows of L that go with them, a piece ahead of their products.
    // The normaliser is summed in four parts, the products in parts of 16 features: against 64 bits the term alone is off by 7.6e-8 of
    // itself at head_dim 128 and 8.0e-8 at 64, on the fp32 kernels before 9.1e-8 and 8.5e-8 (in one chain and parts of 32 features
    // 9.3e-8 and 9.2e-8).
    const float* L = hist.L + (size_t)bh * D * D + (size_t)4 * h * D + f0 + l32;
    const float* z = hist.z + (size_t)bh * D + 4 * h;
    const float* qp = static_cast<const float*>(hist.q_hist) + q_at + 4 * h;
    const size_t trow = (size_t)min(row, n_q - 1) * (D / 2) + 2 * h;
    float den;
    f32x4 dens = {};
    // Workgroups of several groups, with one or two value blocks each, have registers for the query's features, formed once for both
    // sums, and for L a piece ahead; without rotation, whose tables do not fit beside them.  The other form waits for memory every
    // eight key features of L and every 32 of the normaliser.  Selection and attention, that form / this one: 12 heads x 1170 x 2340
    // 59.0 / 56.2 us (four groups), a tenth of the blocks 42.9 / 40.4 (two), 24 heads 94.0 / 92.5, at head_dim 64 12 heads 37.1 / 35.8;
    // off by 3.386e-7 / 3.378e-7 against 64 bits.
    constexpr bool kKeep = ND <= 2 && Sh::WAVES == 2;
    if (kKeep && !hist.cosq) {   // uniform
      constexpr int NI = D / 8, PI = 4 / ND;
      f32x4 x[NI], zz[NI];
      float a[2][PI][4][ND];
      const __amdgpu_buffer_rsrc_t L_rows =
          __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(hist.L + (size_t)bh * D * D), 0, D * D * 4, 0x00020000);
      const int l_at = (4 * h * D + f0 + l32) * 4;
      auto request = [&](int p) {
#pragma unroll
        for (int i = 0; i < PI; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int j = 0; j < ND; ++j)
              a[p & 1][i][e][j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                      L_rows, l_at + (e * D + 32 * j) * 4, 8 * (PI * p + i) * D * 4, 0));
      };
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        x[i] = *reinterpret_cast<const f32x4*>(qp + 8 * i);
        zz[i] = *reinterpret_cast<const f32x4*>(z + 8 * i);
      }
      if (ND == 1) request(0);   // (two blocks' behind z, whose registers they take)
      __builtin_amdgcn_sched_barrier(0);
      auto features = [&](int phi) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            x[i][e] = phi_apply(x[i][e], phi);
            dens[e] = fmaf(x[i][e], zz[i][e], dens[e]);
          }
      };
      if (hist.phi_kind == HF_PHI_RELU) features(HF_PHI_RELU); else features(HF_PHI_ELU1);   // uniform
      if (ND > 1) request(0);
      den = hist.z_scale * both_halves_sum((dens[0] + dens[1]) + (dens[2] + dens[3])) + hist.eps;
      w *= den;
#pragma unroll
      for (int i = 0; i < ND; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[i][r] *= w;
#pragma unroll
      for (int p = 0; p < NI / PI; ++p) {
        if (p + 1 < NI / PI) request(p + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < PI; i += 2) {   // 16 key features, summed for themselves
          f32x16 part[ND];
#pragma unroll
          for (int j = 0; j < ND; ++j) part[j] = {};
#pragma unroll
          for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
              for (int j = 0; j < ND; ++j) part[j] = mfma_f32_wide(a[p & 1][i + u][e][j], x[PI * p + i + u][e], part[j]);
#pragma unroll
          for (int j = 0; j < ND; ++j) o[j] += part[j];
        }
      }
    }
    auto readout = [&](auto relu, auto rotated) {
      auto feature_map = [&](f32x4 x) {
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = phi_apply(x[e], relu.value ? HF_PHI_RELU : HF_PHI_ELU1);
        return x;
      };
#pragma unroll 1
      for (int i0 = 0; i0 < D / 8; i0 += 4) {
        f32x4 x[4], zz[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          x[i] = *reinterpret_cast<const f32x4*>(qp + 8 * (i0 + i));
          zz[i] = *reinterpret_cast<const f32x4*>(z + 8 * (i0 + i));
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          x[i] = feature_map(x[i]);
#pragma unroll
          for (int e = 0; e < 4; ++e) dens[e] = fmaf(x[i][e], zz[i][e], dens[e]);
        }
      }
      den = hist.z_scale * both_halves_sum((dens[0] + dens[1]) + (dens[2] + dens[3])) + hist.eps;
      w *= den;
#pragma unroll
      for (int i = 0; i < ND; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[i][r] *= w;
      constexpr int NB = ND < 2 ? ND : 2;   // value blocks at a time: what four of them need does not fit the registers
#pragma unroll
      for (int j0 = 0; j0 < ND; j0 += NB) {
        f32x4 x[2];
        f32x2 cs[2], sn[2];
        float a[2][4][NB];
        auto request = [&](int i, int u) {
          x[u] = *reinterpret_cast<const f32x4*>(qp + 8 * i);
          if constexpr (rotated.value) {
            cs[u] = *reinterpret_cast<const f32x2*>(hist.cosq + trow + 4 * i);
            sn[u] = *reinterpret_cast<const f32x2*>(hist.sinq + trow + 4 * i);
          }
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int j = 0; j < NB; ++j) a[u][e][j] = L[(size_t)(8 * i + e) * D + 32 * (j0 + j)];
        };
        request(0, 0);
#pragma unroll 1
        for (int i = 0; i < D / 8; i += 2) {   // 16 key features, summed for themselves
          f32x16 part[NB];
#pragma unroll
          for (int j = 0; j < NB; ++j) part[j] = {};
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            if (i + u + 1 < D / 8) request(i + u + 1, u ^ 1);
            f32x4 ph = feature_map(x[u]);
            if constexpr (rotated.value) ph = rotate4(ph, cs[u][0], sn[u][0], cs[u][1], sn[u][1]);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
              for (int j = 0; j < NB; ++j) part[j] = mfma_f32_wide(a[u][e][j], ph[e], part[j]);
          }
#pragma unroll
          for (int j = 0; j < NB; ++j) o[j0 + j] += part[j];
        }
      }
    };
    if (kKeep && !hist.cosq) {
    } else if (hist.phi_kind == HF_PHI_RELU) {   // uniform
      if (kKeep || hist.cosq) readout(std::true_type{}, std::true_type{}); else readout(std::true_type{}, std::false_type{});
    } else {
      if (kKeep || hist.cosq) readout(std::false_type{}, std::true_type{}); else readout(std::false_type{}, std::false_type{});
    }
    w = 1.0f / den;
  }
  // ---- rows through LDS, stored coalesced
  float* const stage = reinterpret_cast<float*>(smem);
#pragma unroll
  for (int i = 0; i < ND; ++i)
#pragma unroll
    for (int rq = 0; rq < 4; ++rq)
      *reinterpret_cast<f32x4*>(stage + (32 * wr + l32) * OST + f0 + 32 * i + 8 * rq + 4 * h) =
          f32x4{o[i][4 * rq], o[i][4 * rq + 1], o[i][4 * rq + 2], o[i][4 * rq + 3]} * w;
  __syncthreads();
  for (int e = tid; e < 32 * RG * (D / 4); e += NT) {
    const int rr = e / (D / 4), c4 = e - rr * (D / 4);
    if (row0 + rr < q_end)
      *reinterpret_cast<f32x4*>(O + ((size_t)bh * n_q + row0 + rr) * D + 4 * c4) = *reinterpret_cast<const f32x4*>(stage + rr * OST + 4 * c4);
  }
}

template <int D, int KG>
int launch_split(const hf_config& c, const void* Q, int n_q, const void* K, const void* V, int n_kv, const int32_t* idx, int k,
                 void* O, const WideHist& hist, hipStream_t s) {
  const int t_m = (n_q + c.block_q - 1) / c.block_q, t_n = (n_kv + c.block_kv - 1) / c.block_kv;
  const int chunks = c.block_q / (32 * RG);
  const long long total = (long long)c.batch * c.heads * t_m * chunks;
  if (total > (1ll << 30)) { set_error("too many query blocks"); return HF_ERR_SHAPE; }
  const int per_xcd = (int)((total + 7) / 8);
  const float scale = c.softmax_scale > 0.0f ? c.softmax_scale : 1.0f / sqrtf((float)D);
  hipLaunchKernelGGL((attn_split_kernel<D, KG>), dim3(8 * per_xcd), dim3(64 * RG * KG), 0, s, static_cast<const float*>(Q),
                     static_cast<const float*>(K), static_cast<const float*>(V), idx, k, n_q, n_kv, kv_stride_of(c, n_kv),
                     c.block_q, c.block_kv, t_m, t_n, chunks, per_xcd, (int)total, scale * 1.4426950408889634f, hist,
                     static_cast<float*>(O));
  return check_launch("hf_hybrid_attn_fwd(attention)");
}

}  // namespace

// The descriptors hold the first key in 24 bits.  Launches of few query rows stay with the kernels in fp32 products, which fill
// the chip with half or a quarter as many rows a workgroup: theirs / the best here, us, head_dim 128: 128 workgroups of 64 rows x 64
// keys 10.2 / 12.3, x 384 21.5 / 27.2, x 1536 60 / 78; 132 x 64 12.8 / 12.3, x 384 32.2 / 27.0, x 1536 96 / 77.  (With the history term
// 19.7 / 20.8 at 132 x 64, 24.2 / 21.2 at 200 x 64; head_dim 64 alike, 6.7 / 7.9 at 128 x 64, 8.2 / 7.8 at 132 x 64.)
bool attn_split_supported(const hf_config& c, int n_q, int n_kv) {
  return c.dtype == HF_F32 && c.block_q % 64 == 0 && c.block_kv % TK == 0 && n_kv < (1 << 23) && row_groups(c, n_q, 64) > 128;
}

// Groups per workgroup: as many as finish in the fewest rounds of the chip (a compute unit has room for eight wavefronts at head_dim
// 128, twelve at 64), of equal ones the fewest where lists are short, whose parts take longer to meet than they save: a round of
// four groups is 256 workgroups, one of two 512 (768), one of one 1024 (1536).  One / two / four groups, us, head_dim 128:
//   workgroups   132               512               520               768              900          1030         1600         2048
//    64 keys     15.5/12.3/16.4    21.2/18.6/31.6    23.3/27.3/45.5    25.2/28.2/47.0   26.4/32.3    37.3/40.6    47.4/53.4    54.2/59.9
//   192          27.0/19.3/21.6    38.9/29.8/42.9    40.5/42.7/62.3    43.8/43.8/63.3   48.3/51.8    66.3/64.1    -            94  /98
//   256          33.4/23.4/22.5    -                 50.1/52.3/63.6    54.2/53.3/65.3   -            82.8/78.8    106 /105     118 /121
//   320          38.4/25.8/26.5    -                 59.4/60.8/80.0    63.9/61.5/81.3   -            -            -            -
//   384          44.2/29.6/27.0    65.5/47.0/54.9    67.4/68.0/79.5    73.0/68.6/81.5   80.5/83.3    112 /104     147 /142     160 /162
//   1536         149 /93  /77      227 /150 /160     231 /218 /231     248 /225 /237    276 /277     392 /347     523 /487     572 /561
// head_dim 64 (one / two): 512 x 64 12.3 / 11.1, 520 x 64 13.3 / 15.6, x 256 28.9 / 29.0, x 384 38.5 / 37.7, x 1536 131 / 121, 780 x 1536
// 143 / 147.  Above, one group is at most 7 % behind on long lists (1700 x 1536 531 / 495 at head_dim 128) and up to a quarter ahead on short ones.
int launch_attn_split(const hf_config& c, const void* Q, int n_q, const void* K, const void* V, int n_kv, const int32_t* idx,
                      int k, void* O, const WideHist& hist, hipStream_t s) {
  const long long wgs = row_groups(c, n_q, 64), keys = idx ? (long long)k * c.block_kv : n_kv;
  if (c.head_dim == 64) {
    if (wgs <= (keys > 256 ? 768 : 512)) return launch_split<64, 2>(c, Q, n_q, K, V, n_kv, idx, k, O, hist, s);
    return launch_split<64, 1>(c, Q, n_q, K, V, n_kv, idx, k, O, hist, s);
  }
  if (wgs <= 256 && keys > 320) return launch_split<128, 4>(c, Q, n_q, K, V, n_kv, idx, k, O, hist, s);
  if (wgs <= (keys > 256 ? 768 : 512) || (wgs > 1024 && wgs <= 1664 && keys > 128)) return launch_split<128, 2>(c, Q, n_q, K, V, n_kv, idx, k, O, hist, s);
  return launch_split<128, 1>(c, Q, n_q, K, V, n_kv, idx, k, O, hist, s);
}

}  // namespace hf
