// Code search by beam search (Appendix C, code optimisation), 8-bit codes, beams of at most 8, plain
// and data-aware: the decisions of k_beam.hip (same binary32 errors in the same stated order, same
// tie-breaks, so the same codes and errors bit for bit), with the matrix cores as a filter.
//
// What bounds it: evaluating a candidate exactly costs 19 to 23 dependent vector instructions and
// a beam of 8 has 2048 candidates per group and stage, of which 8 are kept. Here a candidate's
// error is first approximated on the matrix cores,
//   e = base_p + f_p (sum_t v_pt C_c[t] + s'_p n_c),
// v_p the kept tuple's residual (data-aware: H r) times -2 sign(s) and a power of two, rounded to
// fp16, n_c = |C_c|^2 (C_c^T H C_c) as the sum of two fp16 values, base_p = |r_p|^2 (r_p^T H r_p):
// one v_mfma_f32_32x32x16_f16 gives 32 codewords x 32 kept tuples (slots 0..7 the codeword, slots
// 8, 9 n_c), eight of them every candidate of 32 tuples in 128 registers. An upper bound T of the
// beam-th smallest approximate error is the beam-th smallest of the minima over runs of 16
// candidates; every candidate within T plus twice the approximation's error bound (computed per
// tuple from the roundings actually made) is then evaluated exactly and ranked by (error, tuple):
// about 12 candidates per group instead of 2048. The bound is one-sided and rigorous, so no
// candidate that belongs into the beam is missed. Groups the bound cannot serve (values or
// codebooks that are not finite, more near-ties than the list holds) are searched by the wave
// exhaustively, in the same order of decisions; a zero scale or a weight that is not a number
// decides a group at once.
//
// A wave owns 32 groups (plain: 32 consecutive groups of the matrix; data-aware: 32 rows of one
// group column, which share H) from the first stage to the last: stage 0 has one tuple per group
// (32 groups a pass), later stages PC = beam rounded up to a power of two (32 / PC groups a pass; the
// columns of two passes are prepared at once, one per lane). All state between stages (codes and
// key of every kept tuple) stays in LDS.
//
// Measured (4096 x 4096, k = 4, beam 8): 11.3 ms for the lane-per-group search of k_beam.hip, 2.48 ms
// here; data-aware (2000 x 2304, k = 3, beam 5): 1256 -> 512 us. The bound is still vector issue, busy 70 % of
// the time by the counters (the matrix cores 7 %): a pass (8192 candidates) takes 636 vector
// instructions. By reading, 144 of them are the minima and compares of every candidate, about 170 each
// the threshold and the exact errors, 115 its columns' preparation; the eight MFMAs hide under them.
#include "device.h"
#include "launch.h"

namespace aqmb {

namespace beamf {
constexpr int kWaves = 8;                   // waves per workgroup (fewer where the codebooks need the LDS)
constexpr int kCap = 24;                    // list entries per kept tuple of a pass
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
struct Book { int g, b, bad; float cn, nmax; };   // per codebook: scalings of C and n, max |C'|_2, max |n'|
struct WaveMem {                            // one wave's LDS
  unsigned long long list[32 * kCap];       // candidates: (ordered error, key, p)
  uint16_t quad[32 * kCap];                 // runs of four candidates with one near the threshold: (p, first c)
  uint4 w[32];                              // the groups' weights
  uint2 st[32][8];                          // codes of the kept tuples (byte m = c_m)
  uint16_t ky[32][8];                       // their keys (parent rank << 8 | c); 0xFFFF: none
  float rs[64][12];                         // pass columns: v (8), base, rank, codes
  float s[32], oute[32];
  uint32_t cnt[2][32];
};
struct Args {
  const uint16_t* W;          // [d_out][d_in] fp16
  const uint16_t* codebooks;  // [>= k][256][8] fp16
  const uint16_t* scales;     // [d_out] fp16
  const float* H;             // [G][8][8] fp32 (data-aware)
  unsigned char* codes;       // [k][d_out][G]
  float* errors;              // [d_out][G] or null
  int d_out, d_in, G, k, beam;
  int units, upc;             // 32-group units (data-aware: per group column, upc of them per workgroup)
};
struct Tables {               // the workgroup's LDS tables
  const uint4* books;         // [k][256] codewords times 2^g (fp16)
  const uint32_t* nhl;        // [k][256] n 2^b as two fp16 values
  const float* Q;             // [k][256] C^T H C (data-aware)
  const Book* info;           // [k]
  const float* H;             // the group column's block (data-aware, global memory)
};

__device__ __forceinline__ void wave_sync() {   // LDS writes of the wave's lanes before later reads
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}
__device__ __forceinline__ bool before(float e, uint32_t key, float e2, uint32_t key2) {
  return e < e2 || (e == e2 && key < key2);
}
// Unsigned order of finite floats (-0 as +0) and back.
__device__ __forceinline__ uint32_t ordered(float e) {
  const uint32_t u = __builtin_bit_cast(uint32_t, e + 0.0f);
  return u ^ (uint32_t)(((int32_t)u >> 31) | (int32_t)0x80000000);
}
__device__ __forceinline__ float unordered(uint32_t u) {
  return __builtin_bit_cast(float, u ^ ((u >> 31) ? 0x80000000u : 0xFFFFFFFFu));
}
__device__ __forceinline__ float pow2f(int e) { return __builtin_bit_cast(float, (uint32_t)(e + 127) << 23); }   // |e| <= 126
__device__ __forceinline__ int exp_of(float x) { return (int)((__builtin_bit_cast(uint32_t, x) >> 23) & 0xFFu) - 127; }
__device__ __forceinline__ float fbits(uint32_t u) { return __builtin_bit_cast(float, u); }
__device__ __forceinline__ uint32_t ubits(float f) { return __builtin_bit_cast(uint32_t, f); }

__device__ __forceinline__ void unpack8(const uint4& v, float (&x)[8]) {
  const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    x[2 * q] = f16lo(u[q]);
    x[2 * q + 1] = f16hi(u[q]);
  }
}
// d_t = fma(C_t, m, x_t), C_t the eight fp16 values of v: one rounding. With m C_t exact (two 11-bit
// significands) this is the rounded sum of x_t and the product.
__device__ __forceinline__ void fma8(const uint4& v, float m, const float (&x)[8], float (&d)[8]) {
  const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel_hi:[1,0,0]" : "=v"(d[2 * q]) : "v"(u[q]), "v"(m), "v"(x[2 * q]));
    asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[1,0,0] op_sel_hi:[1,0,0]"
        : "=v"(d[2 * q + 1]) : "v"(u[q]), "v"(m), "v"(x[2 * q + 1]));
  }
}

// fl(sum_u fl(h_u v_u)), u = 0..7 left to right
__device__ __forceinline__ float dot8(const float (&h)[8], const float (&v)[8]) {
#pragma clang fp contract(off)
  float acc = h[0] * v[0];
#pragma unroll
  for (int u = 1; u < 8; ++u) acc = acc + h[u] * v[u];
  return acc;
}

// The exact error of a candidate, in the order stated in k_beam.hip. Plain: v = r, ns2 = -s 2^-g and
// C the codeword times 2^g (their products are those of s and the codeword, exact). Data-aware:
// v = H r, base = r^T H r, q = C^T H C, the codeword unscaled by 2^-g (exact; -0 kept).
template <bool WT>
__device__ __forceinline__ float exact_error(const float (&v)[8], float base, const uint4& C, float s, float ns2, float ginv,
                                             float q) {
#pragma clang fp contract(off)
  if constexpr (WT) {
    float c[8], z[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) z[t] = -0.0f;
    fma8(C, ginv, z, c);
    const float T = dot8(c, v), two_s = 2.0f * s, ss = s * s;
    return (base - two_s * T) + ss * q;
  } else {
    float d[8];
    fma8(C, ns2, v, d);
    return dot8(d, d);
  }
}

__device__ __forceinline__ float min2(float a, float b) { return __builtin_elementwise_minimum(a, b); }
__device__ __forceinline__ float max2(float a, float b) { return __builtin_elementwise_maximum(a, b); }
__device__ __forceinline__ void cswap(float& a, float& b) {
  const float lo = min2(a, b), hi = max2(a, b);
  a = lo;
  b = hi;
}
__device__ __forceinline__ void sort8(float (&m)[8]) {
  cswap(m[0], m[1]); cswap(m[2], m[3]); cswap(m[4], m[5]); cswap(m[6], m[7]);
  cswap(m[0], m[2]); cswap(m[1], m[3]); cswap(m[4], m[6]); cswap(m[5], m[7]);
  cswap(m[1], m[2]); cswap(m[5], m[6]);
  cswap(m[0], m[4]); cswap(m[1], m[5]); cswap(m[2], m[6]); cswap(m[3], m[7]);
  cswap(m[2], m[4]); cswap(m[3], m[5]);
  cswap(m[1], m[2]); cswap(m[3], m[4]); cswap(m[5], m[6]);
}
__device__ __forceinline__ void bitonic8(float (&m)[8]) {   // a bitonic sequence, ascending
  cswap(m[0], m[4]); cswap(m[1], m[5]); cswap(m[2], m[6]); cswap(m[3], m[7]);
  cswap(m[0], m[2]); cswap(m[1], m[3]); cswap(m[4], m[6]); cswap(m[5], m[7]);
  cswap(m[0], m[1]); cswap(m[2], m[3]); cswap(m[4], m[5]); cswap(m[6], m[7]);
}
template <int CTRL> __device__ __forceinline__ float dpp(float x) {
  return fbits((uint32_t)__builtin_amdgcn_update_dpp(0, (int)ubits(x), CTRL, 0xF, 0xF, false));
}
struct Halves { float a, b; };              // a value's copies in the lower and the upper half wave
__device__ __forceinline__ Halves halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(ubits(x), ubits(x), false, false);
  return {fbits((uint32_t)r[0]), fbits((uint32_t)r[1])};
}
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kHalfMirror = 0x141;   // quad_perm, quad_perm, row_half_mirror
// t_i = min(m_i, m_(7-i) of the lane that the DPP pattern names). The waits before a DPP read of a
// register just written are the s_nop (a compiler cannot see into the block).
#define AQMB_MIN8_DPP(PATTERN)                                                                              \
  asm("s_nop 1\n\t"                                                                                          \
      "v_min_f32_dpp %0, %15, %8 " PATTERN " row_mask:0xf bank_mask:0xf\n\t"                                 \
      "v_min_f32_dpp %1, %14, %9 " PATTERN " row_mask:0xf bank_mask:0xf\n\t"                                 \
      "v_min_f32_dpp %2, %13, %10 " PATTERN " row_mask:0xf bank_mask:0xf\n\t"                                \
      "v_min_f32_dpp %3, %12, %11 " PATTERN " row_mask:0xf bank_mask:0xf\n\t"                                \
      "v_min_f32_dpp %4, %11, %12 " PATTERN " row_mask:0xf bank_mask:0xf\n\t"                                \
      "v_min_f32_dpp %5, %10, %13 " PATTERN " row_mask:0xf bank_mask:0xf\n\t"                                \
      "v_min_f32_dpp %6, %9, %14 " PATTERN " row_mask:0xf bank_mask:0xf\n\t"                                 \
      "v_min_f32_dpp %7, %8, %15 " PATTERN " row_mask:0xf bank_mask:0xf"                                     \
      : "=&v"(t[0]), "=&v"(t[1]), "=&v"(t[2]), "=&v"(t[3]), "=&v"(t[4]), "=&v"(t[5]), "=&v"(t[6]), "=&v"(t[7]) \
      : "v"(m[0]), "v"(m[1]), "v"(m[2]), "v"(m[3]), "v"(m[4]), "v"(m[5]), "v"(m[6]), "v"(m[7]))
// The eight smallest of two lanes' sorted lists (the other lane through the DPP pattern), not sorted.
template <int CTRL> __device__ __forceinline__ void merge_dpp(float (&m)[8]) {
  float t[8];
  if constexpr (CTRL == kXor1) AQMB_MIN8_DPP("quad_perm:[1,0,3,2]");
  else if constexpr (CTRL == kXor2) AQMB_MIN8_DPP("quad_perm:[2,3,0,1]");
  else AQMB_MIN8_DPP("row_half_mirror");
#pragma unroll
  for (int i = 0; i < 8; ++i) m[i] = t[i];
}

__device__ __forceinline__ float min8(const float (&m)[8]) {
  return min2(min2(min2(m[0], m[1]), min2(m[2], m[3])), min2(min2(m[4], m[5]), min2(m[6], m[7])));
}
// The keep-th smallest of a group's minima: a lane brings the minima m of its candidates in eight
// blocks of 16 (16 PC minima per group). Coarser blocks need fewer merges here, but the bound is then
// looser and a second round of exact evaluations costs more than it saves (joining the half waves
// first: 2652 -> 2699 us on 4096 x 4096, k = 4, beam 8; four blocks of 64 a column: 3469 us).
template <int PC> __device__ __forceinline__ float kth_smallest(float (&m)[8], int keep) {
  if (keep == 1) {                                  // (uniform) the last stage keeps one tuple
    float t = min8(m);
    if constexpr (PC >= 2) t = min2(t, dpp<kXor1>(t));
    if constexpr (PC >= 4) t = min2(t, dpp<kXor2>(t));
    if constexpr (PC >= 8) t = min2(t, dpp<kHalfMirror>(t));
    const Halves h = halves(t);
    return min2(h.a, h.b);
  }
  sort8(m);
  if constexpr (PC >= 2) {
    merge_dpp<kXor1>(m);
    bitonic8(m);
  }
  if constexpr (PC >= 4) {
    merge_dpp<kXor2>(m);
    bitonic8(m);
  }
  if constexpr (PC >= 8) {
    merge_dpp<kHalfMirror>(m);
    bitonic8(m);
  }
  float lo[8], hi[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const Halves h = halves(m[i]);
    lo[i] = h.a;
    hi[i] = h.b;
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) m[i] = min2(lo[i], hi[7 - i]);
  if (keep == 8)                                    // (uniform)
    return max2(max2(max2(m[0], m[1]), max2(m[2], m[3])), max2(max2(m[4], m[5]), max2(m[6], m[7])));
  bitonic8(m);
  float T = m[0];
#pragma unroll
  for (int i = 1; i < 7; ++i) T = keep > i ? m[i] : T;
  return T;
}
template <int PC> __device__ __forceinline__ float group_max(float t) {   // over the group's columns
  if constexpr (PC >= 2) t = max2(t, dpp<kXor1>(t));
  if constexpr (PC >= 4) t = max2(t, dpp<kXor2>(t));
  if constexpr (PC >= 8) t = max2(t, dpp<kHalfMirror>(t));
  return t;
}

// The kept tuple p of group gl at stage m: codes, rank of its key, v and base of its residual.
struct Tuple { uint2 codes; uint32_t rank; float v[8], base; };
template <bool WT>
__device__ __forceinline__ Tuple load_tuple(const WaveMem& M, const Tables& tb, int m, int gl, int p) {
  Tuple t;
  t.codes = make_uint2(0u, 0u);
  t.rank = 0;
  if (m > 0) {
    t.codes = M.st[gl][p];
    const uint4 kv = *(const uint4*)&M.ky[gl][0];
    const uint32_t k8[4] = {kv.x, kv.y, kv.z, kv.w};
    const uint32_t mine = M.ky[gl][p];
#pragma unroll
    for (int q = 0; q < 4; ++q) t.rank += ((k8[q] & 0xFFFFu) < mine ? 1u : 0u) + ((k8[q] >> 16) < mine ? 1u : 0u);
  }
  const float s = M.s[gl];
  unpack8(M.w[gl], t.v);
  for (int mm = 0; mm < m; ++mm) {                  // r = w - S_0[c_0] - ..., each subtraction rounded
    const uint32_t c = ((mm < 4 ? t.codes.x : t.codes.y) >> (8 * (mm & 3))) & 0xFFu;
    fma8(tb.books[mm * 256 + c], -s * pow2f(-tb.info[mm].g), t.v, t.v);
  }
  if constexpr (WT) {
    float b[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      float h[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) h[u] = tb.H[i * 8 + u];
      b[i] = dot8(h, t.v);
    }
    t.base = dot8(t.v, b);
#pragma unroll
    for (int i = 0; i < 8; ++i) t.v[i] = b[i];
  } else {
    t.base = dot8(t.v, t.v);
  }
  return t;
}
__device__ __forceinline__ void store_row(float* row, const Tuple& t) {
  *(float4*)row = make_float4(t.v[0], t.v[1], t.v[2], t.v[3]);
  *(float4*)(row + 4) = make_float4(t.v[4], t.v[5], t.v[6], t.v[7]);
  *(float4*)(row + 8) = make_float4(t.base, fbits(t.rank), fbits(t.codes.x), fbits(t.codes.y));
}

// Exhaustive search of stage m of group gl by the whole wave, with the decisions of k_beam.hip:
// candidates in the order (error, key), unordered errors never taken, a missing entry is
// (inf, 0xFFFFFFFF) with code 0xFF and no parent. Returns whether one was missing.
// A lane evaluates 32 candidates as (ordered error, key, p) words, all different. The keep smallest lie
// in the keep lanes with the smallest minima: those lanes list theirs up to the keep-th minimum, and the
// listed words (about keep, at most 32 keep) are ranked. Bound: vector issue, two thirds of it the errors.
template <bool WT>
__device__ __noinline__ bool slow_group(WaveMem& M, const Tables& tb, int m, int gl, int n_par, int keep, bool last) {
  const int lane = threadIdx.x & 63;
  const float ginv = pow2f(-tb.info[m].g), s = M.s[gl], ns2 = -s * ginv;
  const uint4* bk = tb.books + m * 256;
  const float* Q = tb.Q + m * 256;
  wave_sync();                                      // the list and the rows are free
  if (lane < n_par) store_row(M.rs[lane], load_tuple<WT>(M, tb, m, gl, lane));
  if (lane == 0) M.cnt[0][0] = 0;
  wave_sync();
  unsigned long long y[32], lm = ~0ull;
#pragma unroll
  for (int p = 0; p < 8; ++p) {
#pragma unroll
    for (int i = 0; i < 4; ++i) y[4 * p + i] = ~0ull;
    if (p < n_par) {                                // (uniform)
      float v[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) v[t] = M.rs[p][t];
      const uint32_t low = (ubits(M.rs[p][9]) << 16) | (uint32_t)(lane << 8) | (uint32_t)p;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float e = exact_error<WT>(v, M.rs[p][8], bk[i * 64 + lane], s, ns2, ginv, WT ? Q[i * 64 + lane] : 0.f);
        y[4 * p + i] = e == e ? ((unsigned long long)ordered(e) << 32) | (low + (uint32_t)(i << 14)) : ~0ull;
        lm = y[4 * p + i] < lm ? y[4 * p + i] : lm;
      }
    }
  }
  M.list[lane] = lm;
  wave_sync();
  int at = 0;                                       // rank of the lane's minimum
#pragma unroll 8
  for (int i = 0; i < 64; ++i) at += M.list[i] < lm ? 1 : 0;
  const unsigned long long kth = __ballot(at == keep - 1 && lm != ~0ull);   // none: all that are ordered
  const int src = kth ? __builtin_ctzll(kth) : 0;
  unsigned long long T = ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(lm >> 32), src) << 32) |
                         (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)lm, src);
  if (!kth) T = ~0ull - 1;
  unsigned long long* list = M.list + 64;           // at most 32 keep <= 256 entries
  if (lm <= T) {
    uint32_t n = 0;
#pragma unroll
    for (int i = 0; i < 32; ++i) n += y[i] <= T ? 1u : 0u;
    uint32_t pos = atomicAdd(&M.cnt[0][0], n);
#pragma unroll
    for (int i = 0; i < 32; ++i)
      if (y[i] <= T) list[pos++] = y[i];
  }
  wave_sync();
  const int total = __builtin_amdgcn_readfirstlane((int)M.cnt[0][0]);
  if (lane < ((-total) & 7)) list[total + lane] = ~0ull;
  if (lane < 8 && lane >= min(total, keep)) {       // missing entries; none kept from `keep` on
    M.ky[gl][lane] = 0xFFFFu;
    if (lane < keep) {
      M.st[gl][lane] = make_uint2(m < 4 ? 0xFFu << (8 * m) : 0u, m < 4 ? 0u : 0xFFu << (8 * (m - 4)));
      if (last) M.oute[gl] = __builtin_inff();
    }
  }
  wave_sync();
  for (int q = lane; q < total; q += 64) {
    const unsigned long long z = list[q];
    int r = 0;
    for (int i = 0; i < total; i += 8) {
#pragma unroll
      for (int h = 0; h < 8; ++h) r += list[i + h] < z ? 1 : 0;
    }
    if (r < keep) {
      const uint32_t lo = (uint32_t)z, key = lo >> 8, c = key & 0xFFu;
      const float* row = M.rs[lo & 0xFFu];
      uint2 nc = make_uint2(ubits(row[10]), ubits(row[11]));
      if (m < 4) nc.x |= c << (8 * m); else nc.y |= c << (8 * (m - 4));
      M.st[gl][r] = nc;
      M.ky[gl][r] = (uint16_t)key;
      if (last) {                                   // again, for the sign of a zero
        float v[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) v[t] = row[t];
        M.oute[gl] = exact_error<WT>(v, row[8], bk[c], s, ns2, ginv, WT ? Q[c] : 0.f);
      }
    }
  }
  wave_sync();
  return total < keep;
}

// y into the ascending list, dropping its last entry.
template <int N> __device__ __forceinline__ void insert(unsigned long long (&l)[N], unsigned long long y) {
  bool lt[N];
#pragma unroll
  for (int q = 0; q < N; ++q) lt[q] = y < l[q];
#pragma unroll
  for (int q = N - 1; q > 0; --q) l[q] = lt[q] ? (lt[q - 1] ? l[q - 1] : y) : l[q];
  l[0] = lt[0] ? y : l[0];
}

// The same exhaustive search for all groups in `left` at once, two lanes per group (even and odd codewords),
// each with a sorted list of (ordered error, key, p) words; the lists are joined at the end. Returns the
// groups with a missing entry. Per group this costs the errors and the insertions, but always for 32 groups;
// slow_group costs about 1000 instructions of its own per group. 2048 x 2048, k = 4, beams 8 / 5 / 2, us, all
// groups left: one NaN in every codebook 18950 / 13050 / 6750 with a wave per group (every minimum by its own
// wave-wide search) -> 4480 / 3320 / 1090, all codewords equal 19100 / 13150 / 6770 -> 4130 / 2980 / 1340, a
// last codebook of zeros at beam 8 2620 -> 1510. The lane-per-group search of k_beam.hip, 8 waves per SIMD
// against 2 here, takes 3020 / 1470 / 510, 1820 / 1070 / 455 and 2990 on these: inputs that tell no codes
// apart do not pay for a second kernel.
template <bool WT, int PC>
__device__ __noinline__ uint32_t slow_unit(WaveMem& M, const Tables& tb, int m, uint32_t left, int n_par, int keep, bool last) {
  const int lane = threadIdx.x & 63, gl = lane & 31, half = lane >> 5;
  const float ginv = pow2f(-tb.info[m].g), s = M.s[gl], ns2 = -s * ginv, inf = __builtin_inff();
  constexpr unsigned long long kNone = 0xFF800000FFFFFFFFull;   // (inf, no key)
  float v[PC][8], base[PC], best = inf;
  uint32_t low[PC];                                 // rank, p of the keys
  unsigned long long l[PC];
  wave_sync();
#pragma unroll
  for (int p = 0; p < PC; ++p) {
    low[p] = 0;
    base[p] = 0.f;
    l[p] = kNone;
    if (p < n_par) {                                // (uniform)
      const Tuple t = load_tuple<WT>(M, tb, m, gl, p);
#pragma unroll
      for (int i = 0; i < 8; ++i) v[p][i] = t.v[i];
      base[p] = t.base;
      low[p] = (t.rank << 16) | (uint32_t)p;
    }
  }
  float thr = inf;                                  // no smaller than the keep-th smallest error of the group
  for (int c0 = half; c0 < 256; c0 += 8) {          // four codewords at a time: four chains of sums in flight
    uint4 C[4];
    float q[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      C[i] = tb.books[m * 256 + c0 + 2 * i];
      q[i] = WT ? tb.Q[m * 256 + c0 + 2 * i] : 0.f;
    }
#pragma unroll
    for (int p = 0; p < PC; ++p)
      if (p < n_par) {
        float e[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) e[i] = exact_error<WT>(v[p], base[p], C[i], s, ns2, ginv, q[i]);
        const float em = __builtin_fminf(__builtin_fminf(e[0], e[1]), __builtin_fminf(e[2], e[3]));
        if (em <= thr) {
          const uint32_t key0 = low[p] + (uint32_t)(c0 << 8);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const uint32_t key = key0 + (uint32_t)(i << 9);
            if (last) {
              const uint32_t at = (uint32_t)l[0];
              const bool bt = before(e[i], key, best, at);
              best = bt ? e[i] : best;
              l[0] = bt ? key : at;
            } else if (e[i] <= thr) {
              const unsigned long long y = ((unsigned long long)ordered(e[i]) << 32) | key;
              if (y < l[PC - 1]) insert<PC>(l, y);
            }
          }
        }
      }
    // Each half has (PC + 1) / 2 errors up to its own bound.
    const Halves h = halves(last ? best : unordered((uint32_t)(l[(PC - 1) / 2] >> 32)));
    thr = last || PC == 1 ? min2(h.a, h.b) : max2(h.a, h.b);
  }
  if (last) l[0] = ((unsigned long long)ordered(best) << 32) | (uint32_t)l[0];
  unsigned long long o[PC];
#pragma unroll
  for (int q = 0; q < PC; ++q) o[q] = __shfl_xor(l[q], 32, 64);
  const float ob = __shfl_xor(best, 32, 64);
  best = o[0] < l[0] ? ob : best;                   // with the sign of a zero
#pragma unroll
  for (int q = 0; q < PC; ++q) insert<PC>(l, o[q]);
  bool missing = false;
  uint2 codes[PC];
#pragma unroll
  for (int q = 0; q < PC; ++q) {
    const uint32_t key = (uint32_t)l[q], c = (key >> 8) & 0xFFu;
    const bool none = key == 0xFFFFFFFFu;           // code 255, no parent
    missing = missing || (none && q < keep);
    codes[q] = make_uint2(0u, 0u);
    if (m > 0 && !none) codes[q] = M.st[gl][key & 7u];
    if (m < 4) codes[q].x |= c << (8 * m); else codes[q].y |= c << (8 * (m - 4));
  }
  wave_sync();                                      // every read of the tuples is done
  if (half == 0 && ((left >> gl) & 1u)) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      if (q < PC && q < keep) M.st[gl][q] = codes[q < PC ? q : 0];
      M.ky[gl][q] = q < PC && q < keep ? (uint16_t)((uint32_t)l[q < PC ? q : 0] >> 8) : (uint16_t)0xFFFFu;
    }
    if (last) M.oute[gl] = best;
  }
  wave_sync();
  return left & (uint32_t)__ballot(missing);
}

// Stage m of the wave's 32 groups, n_par <= PC kept tuples each: the keep best candidates replace
// them. taint: groups with a missing entry so far (bit = group). Returns the groups left to
// slow_group (their tuples unchanged).
template <bool WT, int PC>
__device__ __forceinline__ uint32_t beam_stage(WaveMem& M, const Tables& tb, int m, int n_par, int keep, bool last,
                                               uint32_t taint) {
  constexpr int NCOL = PC == 1 ? 32 : 64, SUB = NCOL / 32;   // columns prepared at once (one per lane), passes on them
  constexpr int NG = 32 / PC, CAP = kCap * PC;               // groups of a pass, list entries per group
  constexpr float kEps = 3.814697265625e-06f;                // 2^-18: sums of at most 18 rounded terms, with room
  const int lane = threadIdx.x & 63, col = lane & 31, half = lane >> 5;
  const uint4* bk = tb.books + m * 256;
  const Book B = tb.info[m];
  const float ginv = pow2f(-B.g), inf = __builtin_inff();
  uint32_t left = 0;
  if (last && lane < 32) M.cnt[0][lane] = 0;
  for (int it = 0; it < 32 * PC / NCOL; ++it) {
    const int cc = lane & (NCOL - 1), p0 = cc % PC, gl0 = it * (NCOL / PC) + cc / PC;
    const bool valid0 = p0 < n_par;
    const Tuple t = load_tuple<WT>(M, tb, m, gl0, valid0 ? p0 : 0);
    if (lane < NCOL) store_row(M.rs[cc], t);
    const float s0 = M.s[gl0], sa = fabsf(s0);
    // Filter operand of the column: 2^a brings the largest 2 |v_t| into [2^12, 2^13) unless that
    // would take s' = |s| 2^(a + g - b) above 2^14.
    float vmax = fabsf(t.v[0]);
#pragma unroll
    for (int i = 1; i < 8; ++i) vmax = max2(vmax, fabsf(t.v[i]));   // NaN if any is
    bool bad = B.bad || !(sa < inf) || s0 == 0.f || !(fabsf(t.base) < 1e30f) || !(vmax < 1e30f);
    const int a_s = 13 - exp_of(sa) - B.g + B.b;
    int a = vmax > 0.f ? min(11 - exp_of(vmax), a_s) : a_s;
    bad = bad || abs(a) > 80 || abs(a + B.g) > 80 || abs(a + B.g - B.b) > 80;
    if (bad) a = 0;
    const float f0 = sa * pow2f(bad ? 0 : -(a + B.g)), sp = sa * pow2f(bad ? 0 : a + B.g - B.b);
    const float sp16 = sp < 6.103515625e-05f ? 0.f : (float)(_Float16)sp;
    const float fac = (s0 < 0.f ? 2.0f : -2.0f) * pow2f(a);
    float x[8], vv = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      x[i] = t.v[i] * fac;
      if constexpr (WT) vv = __builtin_fmaf(x[i], x[i], vv);
    }
    if constexpr (!WT) vv = t.base * (fac * fac);
    // |rounding of v| <= 2^-11 |v| (below the smallest normal: 2^-14 each), of s' as found; sums and
    // every other rounding 2^-18 of the terms' sizes
    const float gm0 = group_max<PC>(
        valid0 ? 1.001f * f0 * ((__builtin_amdgcn_sqrtf(vv) * (4.8828125e-04f + kEps) + 9.765625e-04f) * B.cn +
                                (fabsf(sp - sp16) + kEps * sp) * B.nmax) + kEps * fabsf(t.base)
               : 0.f);
    const uint64_t badcols = __ballot(valid0 && bad);
    const bool slow0 = ((badcols >> (lane & ~(PC - 1))) & ((1ull << PC) - 1)) != 0 || ((taint >> gl0) & 1u);
    const uint32_t hi0[4] = {pack_f16x2(x[0], x[1]), pack_f16x2(x[2], x[3]), pack_f16x2(x[4], x[5]), pack_f16x2(x[6], x[7])};
    const uint32_t sp0 = pack_f16x2(sp16, sp16);
    const float rf0 = __builtin_amdgcn_rcpf(f0), fl0 = slow0 ? 1.0f : valid0 ? 0.0f : 2.0f;
    Halves hx[4], hs, hb, hf, hr, hg, hl;
#pragma unroll
    for (int i = 0; i < 4; ++i) hx[i] = halves(fbits(hi0[i]));
    hs = halves(fbits(sp0)); hb = halves(t.base); hf = halves(f0); hr = halves(rf0); hg = halves(gm0); hl = halves(fl0);
#pragma unroll
    for (int h = 0; h < SUB; ++h) {
      // pass columns 32 h ..: this lane's column is 32 h + col, its candidates the rows of its half
      auto of = [&](const Halves& v) { return h ? v.b : v.a; };
      const int lg = col / PC, p = col % PC, gl = it * (NCOL / PC) + h * NG + lg;
      const float base = of(hb), f = of(hf), rf = of(hr), fl = of(hl);
      const uint32_t sp2 = ubits(of(hs));
      const uint4 bw = make_uint4(half ? sp2 : ubits(of(hx[0])), half ? 0u : ubits(of(hx[1])),
                                  half ? 0u : ubits(of(hx[2])), half ? 0u : ubits(of(hx[3])));
      const f16x8_t bop = __builtin_bit_cast(f16x8_t, bw);
      if (!last && lane < 2 * NG) M.cnt[lane & 1][lane >> 1] = 0;
      // Every candidate of the 32 columns: element e of block blk is codeword 32 blk + 8 (e / 4) + 4 half + e % 4.
      float qm[32];                                  // minima of runs of four codewords
#pragma unroll
      for (int blk = 0; blk < 8; ++blk) {
        uint4 av = bk[blk * 32 + col];
        const uint32_t nv = tb.nhl[m * 256 + blk * 32 + col];
        av.x = half ? nv : av.x;                     // slots 8, 9; slots 10..15 meet zeros
        f32x16_t D;
#pragma unroll
        for (int e = 0; e < 16; ++e) D[e] = 0.f;
        D = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, av), bop, D, 0, 0, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q)
          qm[4 * blk + q] = min2(min2(D[4 * q], D[4 * q + 1]), min2(D[4 * q + 2], D[4 * q + 3]));
      }
      float mn[8];
#pragma unroll
      for (int blk = 0; blk < 8; ++blk) {
        const float z = min2(min2(qm[4 * blk], qm[4 * blk + 1]), min2(qm[4 * blk + 2], qm[4 * blk + 3]));
        mn[blk] = __builtin_fmaf(z, f, fl > 1.5f ? inf : base);
      }
      const float T = kth_smallest<PC>(mn, keep);
      const float te = T + 2.0f * of(hg) + 4.0f * kEps * fabsf(T);
      // the threshold in the column's own units, rounded up
      float thr = (te - base) * rf;
      thr = thr + (4.0f * kEps) * (fabsf(thr) + fabsf(base * rf));
      thr = fl != 0.f ? -inf : thr;
      uint32_t mask = 0;                             // run 0 in the highest bit
#pragma unroll
      for (int q = 0; q < 32; q += 8)
        asm("v_cmp_le_f32 vcc, %1, %9\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc\n\t"
            "v_cmp_le_f32 vcc, %2, %9\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc\n\t"
            "v_cmp_le_f32 vcc, %3, %9\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc\n\t"
            "v_cmp_le_f32 vcc, %4, %9\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc\n\t"
            "v_cmp_le_f32 vcc, %5, %9\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc\n\t"
            "v_cmp_le_f32 vcc, %6, %9\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc\n\t"
            "v_cmp_le_f32 vcc, %7, %9\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc\n\t"
            "v_cmp_le_f32 vcc, %8, %9\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc"
            : "+v"(mask)
            : "v"(qm[q]), "v"(qm[q + 1]), "v"(qm[q + 2]), "v"(qm[q + 3]), "v"(qm[q + 4]), "v"(qm[q + 5]), "v"(qm[q + 6]),
              "v"(qm[q + 7]), "v"(thr)
            : "vcc");
      const uint32_t n = __popc(mask);
      if (last) {                                    // about one run per group: left to last_stage
        if (n > 0) {
          uint32_t at = atomicAdd(&M.cnt[0][gl], n);
          while (mask) {
            const int o = __builtin_clz(mask);
            mask &= ~(0x80000000u >> o);
            if (at < (uint32_t)kCap) M.quad[gl * kCap + at] = (uint16_t)((p << 8) | (32 * (o >> 2) + 8 * (o & 3) + 4 * half));
            ++at;
          }
        }
        uint32_t sm = (uint32_t)__ballot(fl == 1.0f && half == 0 && p == 0);
        while (sm) {
          const int l = __builtin_ctz(sm);
          sm &= sm - 1;
          left |= 1u << (it * (NCOL / PC) + h * NG + l / PC);
        }
        continue;
      }
      wave_sync();
      uint32_t pos = 0;
      if (n > 0) pos = atomicAdd(&M.cnt[0][lg], n);
      wave_sync();
      const uint32_t n_quads = M.cnt[0][lg];
      bool slow = fl == 1.0f || n_quads > (uint32_t)CAP;   // the same in all lanes of a group
      uint16_t* quads = M.quad + lg * CAP;
      if (!slow)
        while (mask) {
          const int o = __builtin_clz(mask);
          mask &= ~(0x80000000u >> o);
          quads[pos++] = (uint16_t)((p << 8) | (32 * (o >> 2) + 8 * (o & 3) + 4 * half));
        }
      wave_sync();
      // Exact errors of the runs' candidates; those up to te (which the keep-th best cannot exceed) are listed.
      const uint32_t u = (uint32_t)(half * PC + p);
      const uint32_t nq = slow ? 0u : n_quads;
      const float s = M.s[gl], ns2 = -s * ginv;
      unsigned long long* list = M.list + lg * CAP;
      for (uint32_t q = u; q < nq; q += 2 * PC) {
        const uint32_t pc = quads[q], pp = pc >> 8, c = pc & 0xFFu;
        const float* row = M.rs[h * 32 + lg * PC + pp];
        const float4 r0 = *(const float4*)row, r1 = *(const float4*)(row + 4);
        const float2 r2 = *(const float2*)(row + 8);
        const float vp[8] = {r0.x, r0.y, r0.z, r0.w, r1.x, r1.y, r1.z, r1.w};
        float e[4];
        uint32_t ne = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          e[i] = exact_error<WT>(vp, r2.x, bk[c + i], s, ns2, ginv, WT ? tb.Q[m * 256 + c + i] : 0.f);
          ne += e[i] <= te ? 1u : 0u;
        }
        uint32_t at = ne ? atomicAdd(&M.cnt[1][lg], ne) : 0u;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (e[i] <= te) {
            if (at < (uint32_t)CAP)
              list[at] = ((unsigned long long)ordered(e[i]) << 32) | ((((ubits(r2.y) << 8) | (c + i)) << 8) | pp);
            ++at;
          }
      }
      wave_sync();
      const uint32_t total = M.cnt[1][lg];
      slow = slow || total > (uint32_t)CAP || total < (uint32_t)keep;
      const uint32_t mine = slow ? 0u : total;
      for (uint32_t i = mine + u; i < ((mine + 7u) & ~7u); i += 2 * PC) list[i] = ~0ull;
      if (u == 0 && !slow) *(uint4*)&M.ky[gl][0] = make_uint4(0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu);
      wave_sync();
      for (uint32_t q = u; q < mine; q += 2 * PC) {
        const unsigned long long y = list[q];
        uint32_t at = 0;
        for (uint32_t i = 0; i < mine; i += 8) {
          unsigned long long z[8];
#pragma unroll
          for (int r = 0; r < 8; ++r) z[r] = list[i + r];
#pragma unroll
          for (int r = 0; r < 8; ++r) at += z[r] < y ? 1u : 0u;
        }
        if (at < (uint32_t)keep) {
          const uint32_t lo = (uint32_t)y, key = lo >> 8, c = key & 0xFFu;
          const float* row = M.rs[h * 32 + lg * PC + (lo & 0xFFu)];
          uint2 nc = make_uint2(ubits(row[10]), ubits(row[11]));
          if (m < 4) nc.x |= c << (8 * m); else nc.y |= c << (8 * (m - 4));
          M.st[gl][at] = nc;
          M.ky[gl][at] = (uint16_t)key;
        }
      }
      wave_sync();
      uint32_t sm = (uint32_t)__ballot(slow && u == 0);
      while (sm) {
        const int l = __builtin_ctz(sm);
        sm &= sm - 1;
        left |= 1u << (it * (NCOL / PC) + h * NG + l / PC);
      }
    }
  }
  return left;
}

// The last stage's decision for the wave's 32 groups from the runs that beam_stage left in M.quad
// (group g: M.cnt[0][g] runs from g kCap on): lane l takes every other run of group l % 32.
// Groups in `left`, and those with too many runs (added to it), are not decided.
template <bool WT>
__device__ __forceinline__ uint32_t last_stage(WaveMem& M, const Tables& tb, int m, uint32_t left) {
  const int lane = threadIdx.x & 63, gl = lane & 31;
  const float ginv = pow2f(-tb.info[m].g), s = M.s[gl], ns2 = -s * ginv;
  wave_sync();
  const uint32_t n = M.cnt[0][gl];
  const bool skip = ((left >> gl) & 1u) || n == 0 || n > (uint32_t)kCap;
  left |= (uint32_t)__ballot(skip);
  float be = __builtin_inff();
  uint32_t bkey = 0xFFFFFFFFu;
  uint2 bc = make_uint2(0u, 0u);
  for (uint32_t q = lane >> 5; q < (skip ? 0u : n); q += 2) {
    const uint32_t pc = M.quad[gl * kCap + q], c = pc & 0xFFu;
    const Tuple t = load_tuple<WT>(M, tb, m, gl, (int)(pc >> 8));
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float e = exact_error<WT>(t.v, t.base, tb.books[m * 256 + c + i], s, ns2, ginv, WT ? tb.Q[m * 256 + c + i] : 0.f);
      const uint32_t key = (t.rank << 8) | (c + i);
      const bool bt = before(e, key, be, bkey);
      be = bt ? e : be;
      bkey = bt ? key : bkey;
      if (bt) bc = t.codes;
    }
  }
  if (m < 4) bc.x |= (bkey & 0xFFu) << (8 * m); else bc.y |= (bkey & 0xFFu) << (8 * (m - 4));
  const float oe = __shfl_xor(be, 32, 64);
  const uint32_t ok = __shfl_xor(bkey, 32, 64);
  wave_sync();                                        // every read of the tuples is done
  if (!skip && (before(be, bkey, oe, ok) || (lane < 32 && !before(oe, ok, be, bkey)))) {
    M.st[gl][0] = bc;
    M.oute[gl] = be;
  }
  wave_sync();
  return left;
}

template <bool WT, int PCB>
__global__ __launch_bounds__(64 * kWaves) void beam_mma_kernel(Args a) {
  extern __shared__ uint4 smem_bm[];
  WaveMem* mem = (WaveMem*)smem_bm;
  const int n_waves = blockDim.x >> 6, kThreads = blockDim.x;
  uint4* books = (uint4*)(mem + n_waves);              // [k][256] codewords times 2^g (fp16)
  uint32_t* nhl = (uint32_t*)(books + a.k * 256);     // [k][256] n 2^b as two fp16 values
  float* Qs = (float*)(nhl + a.k * 256);              // [k][256] C^T H C (data-aware)
  __shared__ Book info[8];
  __shared__ uint32_t mx[8][3];                       // maxima (float bits): |C_t|, |C|^2, |n|
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_chunks = WT ? (a.units + a.upc - 1) / a.upc : 1;
  const int j = WT ? blockIdx.x / n_chunks : 0;
  const float* H = WT ? a.H + (size_t)j * 64 : nullptr;
  if (tid < 24) mx[tid / 3][tid % 3] = 0;
  __syncthreads();
  for (int q = tid; q < a.k * 256; q += kThreads) {
    const uint4 raw = ((const uint4*)a.codebooks)[q];
    float c[8], top = 0.f;
    unpack8(raw, c);
    uint32_t nonfinite = 0;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      top = fmaxf(top, fabsf(c[t]));
      nonfinite |= !(fabsf(c[t]) < 1e30f);
    }
    const float c2 = dot8(c, c);
    float n = c2;
    if constexpr (WT) {
      float hc[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        float h[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) h[u] = H[t * 8 + u];
        hc[t] = dot8(h, c);
      }
      n = dot8(c, hc);
      Qs[q] = n;
    }
    books[q] = raw;
    const float na = fabsf(n);
    atomicMax(&mx[q >> 8][0], nonfinite ? 0x7F800000u : __builtin_bit_cast(uint32_t, top));
    atomicMax(&mx[q >> 8][1], nonfinite ? 0x7F800000u : __builtin_bit_cast(uint32_t, c2));
    atomicMax(&mx[q >> 8][2], !(na < 1e30f) ? 0x7F800000u : __builtin_bit_cast(uint32_t, na));
    ((float*)nhl)[q] = n;
  }
  __syncthreads();
  if (tid < a.k) {
    const float top = __builtin_bit_cast(float, mx[tid][0]), c2 = __builtin_bit_cast(float, mx[tid][1]),
                nm = __builtin_bit_cast(float, mx[tid][2]);
    Book B;
    B.bad = !(top < 1e30f) || !(nm < 1e30f);
    B.g = !B.bad && top > 0.f ? max(0, 13 - exp_of(top)) : 0;
    B.b = !B.bad && nm > 1e-30f ? 13 - exp_of(nm) : 0;
    B.cn = B.bad ? 0.f : 1.001f * __builtin_amdgcn_ldexpf(__builtin_amdgcn_sqrtf(c2), B.g);
    B.nmax = B.bad ? 0.f : __builtin_amdgcn_ldexpf(nm, B.b) + 1.0f;
    info[tid] = B;
  }
  __syncthreads();
  for (int q = tid; q < a.k * 256; q += kThreads) {
    const Book B = info[q >> 8];
    float c[8];
    unpack8(books[q], c);
#pragma unroll
    for (int t = 0; t < 8; ++t) c[t] = __builtin_amdgcn_ldexpf(c[t], B.g);   // exact: at most 2^14, or g = 0
    books[q] = make_uint4(pack_f16x2(c[0], c[1]), pack_f16x2(c[2], c[3]), pack_f16x2(c[4], c[5]), pack_f16x2(c[6], c[7]));
    const float n = __builtin_amdgcn_ldexpf(((const float*)nhl)[q], B.b);
    const _Float16 hi = (_Float16)n;
    nhl[q] = B.bad ? 0u : pack_f16x2((float)hi, n - (float)hi);
  }
  __syncthreads();

  WaveMem& M = mem[wave];
  const Tables tb{books, nhl, Qs, info, H};
  const size_t total = (size_t)a.d_out * a.G;
  int u0, u1, du;
  if (WT) {
    u0 = (blockIdx.x % n_chunks) * a.upc + wave;
    u1 = min((int)(blockIdx.x % n_chunks + 1) * a.upc, a.units);
    du = n_waves;
  } else {
    u0 = blockIdx.x * n_waves + wave;
    u1 = a.units;
    du = gridDim.x * n_waves;
  }
  for (int unit = u0; unit < u1; unit += du) {
    const size_t idx = (size_t)unit * 32 + (lane & 31);
    const bool ok = idx < (WT ? (size_t)a.d_out : total);
    const size_t ic = ok ? idx : (WT ? (size_t)a.d_out : total) - 1;
    const size_t row = WT ? ic : ic / (size_t)a.G;
    const size_t o = WT ? ic * a.G + j : ic;          // (row, group) flattened: also the weights' group
    if (lane < 32) {
      M.w[lane] = *(const uint4*)(a.W + o * 8);
      M.s[lane] = f16_to_f32(a.scales[row]);
    }
    wave_sync();
    // Groups that the filter cannot serve: a zero scale, weights or a scale that are not finite. With a zero
    // scale and all else finite every candidate has the error of code 0, which comes first; with a weight that
    // is not a number no candidate has one, and every stage's entries are missing.
    uint32_t taint = 0, done, hopeless;
    {
      const uint4 w = M.w[lane & 31];
      const float s = M.s[lane & 31];
      typedef uint16_t u16x2_t __attribute__((ext_vector_type(2)));
      const u16x2_t mask = {0x7FFF, 0x7FFF};
      auto mag = [&](uint32_t u) { return __builtin_bit_cast(u16x2_t, u) & mask; };
      const u16x2_t top2 = __builtin_elementwise_max(__builtin_elementwise_max(mag(w.x), mag(w.y)),
                                                     __builtin_elementwise_max(mag(w.z), mag(w.w)));
      const uint32_t top = top2[0] > top2[1] ? top2[0] : top2[1];   // the largest magnitude's bits
      const bool nan = top > 0x7C00u, inf = top == 0x7C00u;
      hopeless = (uint32_t)__ballot(top >= 0x7C00u || s == 0.f || !(fabsf(s) < 1e30f));
      done = 0;
      if (hopeless) {                                // (uniform)
        const Tuple t = load_tuple<WT>(M, tb, 0, lane & 31, 0);
        bool zero = s == 0.f && fabsf(t.base) < 1e30f && !inf && !nan;
#pragma unroll
        for (int i = 0; i < 8; ++i) zero = zero && fabsf(t.v[i]) < 1e30f;
        for (int m = 0; m < a.k; ++m) zero = zero && !info[m].bad;
        done = (uint32_t)__ballot(zero || nan);
        if (lane < 32 && (zero || nan)) {
          const int m = a.k - 1;
          const float ginv = pow2f(-info[m].g);
          const uint32_t c = nan ? 0xFFu : 0u;
          M.st[lane][0] = make_uint2(m < 4 ? c << (8 * m) : 0u, m < 4 ? 0u : c << (8 * (m - 4)));
          M.oute[lane] = nan ? __builtin_inff()
                             : exact_error<WT>(t.v, t.base, books[m * 256], s, -s * ginv, ginv, WT ? Qs[m * 256] : 0.f);
        }
        wave_sync();
      }
    }
    for (int m = 0; m < a.k && done != ~0u; ++m) {
      const bool last = m == a.k - 1;
      const int n_par = m == 0 ? 1 : a.beam, keep = last ? 1 : a.beam;
      uint32_t left = ~0u;
      if (!info[m].bad && (taint | hopeless) != ~0u) {   // else the filter serves none of them
        left = m == 0 ? beam_stage<WT, 1>(M, tb, m, n_par, keep, last, taint)
                      : beam_stage<WT, PCB>(M, tb, m, n_par, keep, last, taint);
        if (last) left = last_stage<WT>(M, tb, m, left);
      }
      left = __builtin_amdgcn_readfirstlane(left & ~done);
      // slow_unit: 32 candidates per tuple and group of about 28 instructions; slow_group: 1000 and 4 per tuple
      if (__builtin_popcount(left) >= 2 + 3 * n_par) {
        taint |= slow_unit<WT, PCB>(M, tb, m, left, n_par, keep, last);
        left = 0;
      }
      while (left) {
        const int gl = __builtin_ctz(left);
        left &= left - 1;
        if (slow_group<WT>(M, tb, m, gl, n_par, keep, last)) taint |= 1u << gl;
      }
      taint = __builtin_amdgcn_readfirstlane(taint);
    }
    if (ok) {
      const uint2 cd = M.st[lane & 31][0];
      for (int m = lane >> 5; m < a.k; m += 2)
        a.codes[(size_t)m * total + o] = (unsigned char)(((m < 4 ? cd.x : cd.y) >> (8 * (m & 3))) & 0xFFu);
      if (a.errors && lane < 32) a.errors[o] = M.oute[lane];
    }
    wave_sync();
  }
}

// Waves per workgroup: eight, or what the LDS holds beside the codebook tables (k = 8, data-aware: 7).
static int n_waves(int k, bool weighted) {
  const size_t room = 163840 - 1024 - (size_t)k * 256 * (weighted ? 24 : 20);
  const int w = (int)(room / sizeof(WaveMem));
  return w < kWaves ? w : kWaves;
}

template <bool WT, int PCB>
static hipError_t launch(const Args& a, int grid, hipStream_t st) {
  const int nw = n_waves(a.k, WT);
  const size_t lds = sizeof(WaveMem) * nw + (size_t)a.k * 256 * (WT ? 24 : 20);
  beam_mma_kernel<WT, PCB><<<grid, 64 * nw, lds, st>>>(a);
  return hipGetLastError();
}
template <bool WT>
static hipError_t launch_pc(const Args& a, int grid, hipStream_t st) {
  if (a.beam == 1) return launch<WT, 1>(a, grid, st);
  if (a.beam == 2) return launch<WT, 2>(a, grid, st);
  if (a.beam <= 4) return launch<WT, 4>(a, grid, st);
  return launch<WT, 8>(a, grid, st);
}
}  // namespace beamf

hipError_t launch_beam_mma(const aqmb_desc& d, int k, int beam_width, const void* W, const uint16_t* codebooks,
                           const uint16_t* scales, const float* H, unsigned char* codes, float* errors, hipStream_t st) {
  using namespace beamf;
  Args a{};
  a.W = (const uint16_t*)W;
  a.codebooks = codebooks;
  a.scales = scales;
  a.H = H;
  a.codes = codes;
  a.errors = errors;
  a.d_out = d.d_out;
  a.d_in = d.d_in;
  a.G = d.d_in / d.group_size;
  a.k = k;
  a.beam = beam_width;
  int dev = 0, n_cu = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if ((e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
  if (n_cu < 1) n_cu = 256;
  if (H) {
    a.units = (a.d_out + 31) / 32;
    // Units per wave: the fewest rounds of workgroups (one per compute unit), a workgroup's tables
    // (C^T H C of every codeword) counted as 0.15 unit (2000 x 2304, k = 3, beam 5: one unit a wave,
    // 9 rounds of 256 workgroups, against 5 rounds of two units).
    double best = 0;
    for (int w = 1; w <= 4; ++w) {
      const long long wgs = (long long)((a.units + n_waves(k, true) * w - 1) / (n_waves(k, true) * w)) * a.G;
      const double cost = (double)((wgs + n_cu - 1) / n_cu) * (w + 0.15);
      if (w == 1 || cost < best) { best = cost; a.upc = n_waves(k, true) * w; }
    }
    const int n_chunks = (a.units + a.upc - 1) / a.upc;
    return launch_pc<true>(a, n_chunks * a.G, st);
  }
  a.units = (int)(((size_t)a.d_out * a.G + 31) / 32);
  const int nw = n_waves(k, false), need = (a.units + nw - 1) / nw;
  return launch_pc<false>(a, need < n_cu ? need : n_cu, st);
}

}  // namespace aqmb
