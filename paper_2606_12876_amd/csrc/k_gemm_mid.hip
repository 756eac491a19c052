// Prefill GEMM for tens to hundreds of tokens (8- and 4-bit codes, k <= 4): Y[n][i] = s_i sum_t X[n][t]
// Wb_k[i][t] with Wb_k = RNE_bf16(binary32 left fold of C_m[b_{ijm}] over m < k), bf16 matrix cores,
// fp32 sums: the arithmetic of the other GEMM kernels.
//
// A workgroup of 8 or 16 waves owns 16 RB weight rows and up to 16 NB tokens and splits d_in over its
// waves in runs of 128 inputs (one 16-byte code slice per row and plane). No wave waits for another
// inside the walk: each streams its own part of X through a private LDS ring (a unit is 16 tokens x
// 64 inputs: two direct global->LDS loads of eight full 128-byte lines, two or four units ahead), its
// code slices through a private LDS buffer (one run ahead), and dequantizes the weight fragments of
// the two K-steps of a 64-input chunk into registers, where every token block of the tile uses them.
// Within a chunk lane l stands for weight row (token) l % 16 and groups 2 (l / 16), 2 (l / 16) + 1,
// so its two codes are neighbouring bytes. The partial tiles are added in wave order at the end.
//
// Why: the 16-row tiling reads X fragments straight from memory (16 rows x 64 bytes an instruction:
// 30-36 bytes/clk per CU against 52 for full lines) and re-gathers every weight per 64 tokens; the
// large tiles leave compute units idle below about 2000 tokens and gather each weight from one
// unreplicated codebook copy behind a barrier per 64 inputs. Measured (4096 x 4096, k = 4): 64 tokens
// 23.0 -> 13.3 us, 150: 52.1 -> 20.1, 512: 53 -> 34, 1024: 76 -> 61; 11008 x 4096, k = 3, 333 tokens:
// 75 -> 58 us; 3000 x 11008, k = 2, 100 tokens: 75 -> 22 us. Bound: at few tokens the start and end
// (about 6 us), then X through the CU's L2 port (16 tokens of 4096 inputs in 1.2-1.6 us, two thirds of
// the full-line rate); on the 48- and 64-row tiles the LDS pipe (unit writes and reads beside the
// codeword gathers). Sixteen waves instead of eight: 14.5 -> 13.1 us at 64 tokens, 30 -> 24 us at 100
// tokens of 11008 inputs; a deeper ring changes nothing there.
#include "device.h"
#include "launch.h"

namespace aqmb {

namespace gmid {
constexpr int kUnit = 2048;                                  // bytes of a ring unit
// Waves per workgroup: 16 where the accumulators leave room (16 RB x 16 NB values a wave in 128 registers).
template <int RB, int NB> constexpr int n_waves() { return RB * NB <= 16 ? 16 : 8; }
// Ring units per wave: 4 KiB in flight from each of 16 waves, 8 KiB from each of 8.
template <int RB, int NB> constexpr int depth() { return n_waves<RB, NB>() == 16 ? 2 : 4; }
constexpr int kLds = 163840;
typedef __bf16 b16x8_t __attribute__((ext_vector_type(8)));
// Code bytes a wave keeps: RB 16 rows x K planes x 16 bytes, in whole loads of 1 KiB.
template <int K, int RB> constexpr int code_loads() { return (RB * 16 * K + 63) / 64; }
// Codebook copies: as many as fit beside the rings (16-codeword books fill the banks once: one).
template <int K, int CB, int RB, int NB> constexpr int nrep() {
  if (CB == 4) return 1;
  const int room = kLds - n_waves<RB, NB>() * (depth<RB, NB>() * kUnit + code_loads<K, RB>() * 1024);
  return room >= K * 4096 * 8 ? 8 : room >= K * 4096 * 4 ? 4 : room >= K * 4096 * 2 ? 2 : 1;
}
template <int K, int CB, int RB, int NB> constexpr size_t lds_bytes() {
  return (size_t)n_waves<RB, NB>() * (depth<RB, NB>() * kUnit + code_loads<K, RB>() * 1024) +
         (size_t)K * (1 << CB) * 16 * nrep<K, CB, RB, NB>();
}
struct Args {
  const unsigned char* codes;
  const uint16_t* codebooks;
  const uint16_t* scales;
  const uint16_t* X;          // [n][d_in] bf16
  void* Y;                    // [n][d_out]
  const void* zero_page;
  size_t plane_bytes;
  int d_out, d_in, G, n, y_dtype;
  int nb, n_tt;               // token blocks per tile (<= NB), token tiles
};

// binary32 left fold of K codewords, rounded once to bf16
template <int K> __device__ __forceinline__ b16x8_t fold(const uint4 (&c)[K]) {
  float w[8];
  if constexpr (K == 1) {
    const uint32_t u[4] = {c[0].x, c[0].y, c[0].z, c[0].w};
#pragma unroll
    for (int q = 0; q < 4; ++q) { w[2 * q] = f16lo(u[q]); w[2 * q + 1] = f16hi(u[q]); }
  } else {                                                   // planes 0 and 1 in one step: their sum rounded once
    const uint32_t u[4] = {c[0].x, c[0].y, c[0].z, c[0].w}, v[4] = {c[1].x, c[1].y, c[1].z, c[1].w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel_hi:[1,0,1]" : "=v"(w[2 * q]) : "v"(v[q]), "v"(u[q]));
      asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel:[1,0,1] op_sel_hi:[1,0,1]" : "=v"(w[2 * q + 1]) : "v"(v[q]), "v"(u[q]));
    }
  }
#pragma unroll
  for (int m = 2; m < K; ++m) {
    w[0] = add_f16_lo(c[m].x, w[0]); w[1] = add_f16_hi(c[m].x, w[1]);
    w[2] = add_f16_lo(c[m].y, w[2]); w[3] = add_f16_hi(c[m].y, w[3]);
    w[4] = add_f16_lo(c[m].z, w[4]); w[5] = add_f16_hi(c[m].z, w[5]);
    w[6] = add_f16_lo(c[m].w, w[6]); w[7] = add_f16_hi(c[m].w, w[7]);
  }
  return __builtin_bit_cast(b16x8_t, make_uint4(pack_bf16x2(w[0], w[1]), pack_bf16x2(w[2], w[3]),
                                                pack_bf16x2(w[4], w[5]), pack_bf16x2(w[6], w[7])));
}
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

template <int K, int CB, int RB, int NB>
__global__ __launch_bounds__(64 * (RB * NB <= 16 ? 16 : 8)) void gemm_mid_kernel(Args a) {
  constexpr int kWaves = n_waves<RB, NB>(), kThreads = 64 * kWaves, kR = depth<RB, NB>();
  constexpr int NCW = 1 << CB, kNrep = nrep<K, CB, RB, NB>(), kCL = code_loads<K, RB>();
  constexpr int kShift = kNrep == 8 ? 7 : kNrep == 4 ? 6 : kNrep == 2 ? 5 : 4;
  extern __shared__ uint4 smem_gm[];
  char* smem = (char*)smem_gm;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  char* ring = smem + wave * (kR * kUnit + kCL * 1024);      // this wave's units, then its code slices
  char* cbuf = ring + kR * kUnit;
  char* books = smem + kWaves * (kR * kUnit + kCL * 1024);
  const uint32_t ring_a = lds_addr(ring), cbuf_a = lds_addr(cbuf);
  const int r16 = lane & 15, kc = lane >> 4;
  // Workgroup w runs on XCD w mod 8. Tile by tile, a token tile's workgroups share an XCD only where the
  // number of token tiles and 8 have a common factor; otherwise every XCD walks all of X and its L2
  // holds none of it. There each XCD takes a contiguous range of the tiles instead, row block by row block
  // within a token tile (260 shapes: 1.5 x as fast at odd numbers of token tiles from 11 on, 1.2 at 14 and
  // 18, 1.1 at 5 and 7; the same at multiples of 4).
  int tile = blockIdx.x;                                     // in the plain order
  if (a.n_tt > 2 && (a.n_tt & 3)) {
    const int T = gridDim.x, n_rb = T / a.n_tt, xcd = blockIdx.x & 7;
    const int t = xcd * (T >> 3) + (xcd < (T & 7) ? xcd : (T & 7)) + (int)(blockIdx.x >> 3);
    tile = t % n_rb * a.n_tt + t / n_rb;
  }
  const int tt = tile % a.n_tt, row0 = (tile / a.n_tt) * 16 * RB;
  const int nb = a.nb, t0 = tt * 16 * nb;
  const int n_runs = (a.G + 15) / 16;
  const int mine = (n_runs - wave + kWaves - 1) / kWaves;    // runs of this wave (may be 0)
  // Workgroups start their walk at different runs, so that they read different parts of X at a time.
  const int rot = (int)((blockIdx.x * 5u) % (uint32_t)n_runs);
  auto run_of = [&](int i) { const int r = wave + i * kWaves + rot; return r >= n_runs ? r - n_runs : r; };

  auto load_codes = [&](int i) {                             // code slices of the wave's run i (past the end: the last)
    const int run = run_of(i < mine ? i : (mine > 0 ? mine - 1 : 0));
    const int slice = CB == 8 ? run : run >> 1;
#pragma unroll
    for (int q = 0; q < kCL; ++q) {
      int combo = q * 64 + lane;
      if (combo >= RB * 16 * K) combo = RB * 16 * K - 1;
      const int m = combo / (RB * 16), r = row0 + combo % (RB * 16);
      load_lds16(a.codes + m * a.plane_bytes + ((size_t)slice * a.d_out + (r < a.d_out ? r : a.d_out - 1)) * 16,
                 cbuf_a + q * 1024);
    }
  };
  // Unit u of the wave: run u / (2 nb), chunk (u / nb) % 2, token block u % nb. A load covers 8 tokens
  // x 128 bytes; the 16-byte pieces of a token are swizzled by (token / 2) % 8. The walk's position is
  // kept in three counters (units past the end repeat the last run: their loads are never read).
  int lb = 0, lslot = 0, lch = 0, li = 0;
  const uint32_t row_b = (uint32_t)a.d_in * 2;                // bytes of a token (at most 2^21, see gemm_mid_us)
  const char* Xt = (const char*)(a.X + (size_t)t0 * a.d_in);  // the tile's first token
  const uint32_t last_row = gemm_mid_last_row(a.n, t0, nb);   // tokens past the last read it again, never stored
  uint32_t off0[2], off_max[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint32_t tr = h * 8 + (lane >> 3), piece = (lane & 7) ^ ((tr >> 1) & 7);
    off0[h] = gemm_mid_x_offset(tr, row_b, piece);
    off_max[h] = gemm_mid_x_offset(last_row, row_b, piece);
  }
  int lk0 = mine > 0 ? run_of(0) * 128 : 0;
  uint32_t lrow = 0;                                          // lb * 16 * row_b
  auto load_unit = [&]() {
    const uint32_t dst = ring_a + lslot * kUnit;
    const char* base = Xt + (size_t)lk0 * 2;
    if (lk0 + 64 <= a.d_in) {
#pragma unroll
      for (int h = 0; h < 2; ++h) load_lds16_off(base, min(off0[h] + lrow, off_max[h]), dst + h * 1024);
    } else {                                                  // the ragged last chunk: zeros past d_in
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t piece = (lane & 7) ^ (((h * 8 + (lane >> 3)) >> 1) & 7);
        load_lds16(lk0 + (int)piece * 8 < a.d_in ? (const void*)(base + min(off0[h] + lrow, off_max[h])) : a.zero_page,
                   dst + h * 1024);
      }
    }
    lslot = (lslot + 1) & (kR - 1);
    lrow += 16 * row_b;
    if (++lb == nb) {
      lb = 0;
      lrow = 0;
      lk0 += 64;
      if (++lch == 2) { lch = 0; ++li; lk0 = run_of(li < mine ? li : mine - 1) * 128; }
    }
  };

  if (mine > 0) {
    load_codes(0);
#pragma unroll
    for (int u = 0; u < kR; ++u) load_unit();
  }
  for (int q = tid; q < K * NCW; q += kThreads) {
    const uint4 v = ((const uint4*)a.codebooks)[q];
    const int sw = q >> (8 - kShift);
#pragma unroll
    for (int i = 0; i < kNrep; ++i) *(uint4*)(books + (size_t)(q * kNrep + ((i + sw) & (kNrep - 1))) * 16) = v;
  }
  __syncthreads();

  f32x4_t acc[RB][NB];
#pragma unroll
  for (int r = 0; r < RB; ++r)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[r][b] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const uint32_t rep_off = (uint32_t)(lane & (kNrep - 1)) * 16;
  int slot = 0;
  auto read_unit = [&](b16x8_t (&x)[2]) {                    // the next unit's fragments; then its slot is refilled
    const char* u = ring + slot * kUnit + r16 * 128;
    const int sw = (r16 >> 1) & 7;
    x[0] = *(const b16x8_t*)(u + ((2 * kc) ^ sw) * 16);
    x[1] = *(const b16x8_t*)(u + ((2 * kc + 1) ^ sw) * 16);
    slot = (slot + 1) & (kR - 1);
  };
#pragma unroll 1
  for (int i = 0; i < mine; ++i) {
    const int run = run_of(i);
    // The run's code slices (older than the first unit's loads when a chunk has at least kR units).
    if (nb >= kR - 1) wait_vmcnt<2 * (kR - 1)>(); else wait_vmcnt<0>();
    uint32_t code[2][RB][K];                                  // two codes of this lane per chunk
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int m = 0; m < K; ++m) {
          const char* p = cbuf + (m * RB * 16 + r * 16 + r16) * 16;
          code[c][r][m] = CB == 8 ? *(const uint16_t*)(p + c * 8 + 2 * kc)
                                  : *(const unsigned char*)(p + (run & 1) * 8 + c * 4 + kc);
        }
    wait_lds();
    load_codes(i + 1);
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      b16x8_t w[RB][2];
#pragma unroll
      for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          uint4 cw[K];
#pragma unroll
          for (int m = 0; m < K; ++m) {
            const uint32_t cd = CB == 8 ? (code[c][r][m] >> (8 * j)) & 0xFFu : (code[c][r][m] >> (4 * j)) & 15u;
            cw[m] = *(const uint4*)(books + (((uint32_t)(m * NCW) + cd) << kShift) + rep_off);
          }
          w[r][j] = fold<K>(cw);
        }
      if (run * 16 + 16 > a.G) {                              // (uniform) the ragged last run: the groups past d_in are padding
#pragma unroll                                                // of code 0; zero weights, as codeword 0 may not be finite
        for (int j = 0; j < 2; ++j)
          if (run * 16 + c * 8 + 2 * kc + j >= a.G)
#pragma unroll
            for (int r = 0; r < RB; ++r) w[r][j] = __builtin_bit_cast(b16x8_t, make_uint4(0, 0, 0, 0));
      }
      b16x8_t x0[2], x1[2];
      wait_vmcnt<2 * (kR - 1)>();
      read_unit(x0);
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        if (b < nb) {
          b16x8_t (&cur)[2] = (b & 1) ? x1 : x0;
          b16x8_t (&nxt)[2] = (b & 1) ? x0 : x1;
          wait_lds();                                        // this unit is in registers: refill its slot
          load_unit();
          if (b + 1 < nb) {
            wait_vmcnt<2 * (kR - 1)>();
            read_unit(nxt);
          }
#pragma unroll
          for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int j = 0; j < 2; ++j)
              acc[r][b < NB ? b : 0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[r][j], cur[j], acc[r][b < NB ? b : 0], 0, 0, 0);
        }
      }
    }
  }
  wait_vmcnt<0>();                                            // no load may land in LDS below
  // Partial tiles in wave order; element e of lane l is weight row 4 (l / 16) + e of its 16, token l % 16.
  constexpr int kFit = (int)(lds_bytes<K, CB, RB, NB>() / (kWaves * 1024)), kPer = kFit < RB * NB ? kFit : RB * NB;   // tiles a round
  f32x4_t* red = (f32x4_t*)smem;                              // [kPer][kWaves][64]
  const bool vec = (a.d_out & 3) == 0;
#pragma unroll
  for (int q0 = 0; q0 < RB * NB; q0 += kPer) {
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPer; ++q)
      if (q0 + q < RB * NB) red[(q * kWaves + wave) * 64 + lane] = acc[(q0 + q) % RB][(q0 + q) / RB];
    __syncthreads();
#pragma unroll 1
    for (int q = wave; q < kPer && q0 + q < RB * NB; q += kWaves) {
      const int r = (q0 + q) % RB, b = (q0 + q) / RB;
      const int row = row0 + r * 16 + 4 * kc, t = t0 + b * 16 + r16;
      if (b >= nb) continue;
      f32x4_t sum = red[q * kWaves * 64 + lane];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) sum += red[(q * kWaves + w) * 64 + lane];
      if (t >= a.n || row >= a.d_out) continue;
      const size_t o = (size_t)t * a.d_out + row;
      if (vec) {                                              // four rows at once
        const uint2 sc = *(const uint2*)(a.scales + row);
        const float v0 = sum[0] * f16lo(sc.x), v1 = sum[1] * f16hi(sc.x), v2 = sum[2] * f16lo(sc.y), v3 = sum[3] * f16hi(sc.y);
        if (a.y_dtype == AQMB_BF16) *(uint2*)((uint16_t*)a.Y + o) = make_uint2(pack_bf16x2(v0, v1), pack_bf16x2(v2, v3));
        else *(float4*)((float*)a.Y + o) = make_float4(v0, v1, v2, v3);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (row + e < a.d_out) {
            const float v = sum[e] * f16_to_f32(a.scales[row + e]);
            if (a.y_dtype == AQMB_BF16) OutT<AQMB_BF16>::store(a.Y, o + e, v);
            else OutT<AQMB_F32>::store(a.Y, o + e, v);
          }
      }
    }
  }
}

template <int K, int CB, int RB, int NB>
static hipError_t launch(const Args& a, hipStream_t st) {
  const int grid = ((a.d_out + 16 * RB - 1) / (16 * RB)) * a.n_tt;
  gemm_mid_kernel<K, CB, RB, NB><<<grid, 64 * n_waves<RB, NB>(), lds_bytes<K, CB, RB, NB>(), st>>>(a);
  return hipGetLastError();
}

template <int K, int CB>
static hipError_t launch_shape(Args& a, int rb, int nb_max, hipStream_t st) {
  switch (rb * 100 + nb_max) {
    case 102: return launch<K, CB, 1, 2>(a, st);
    case 104: return launch<K, CB, 1, 4>(a, st);
    case 202: return launch<K, CB, 2, 2>(a, st);
    case 204: return launch<K, CB, 2, 4>(a, st);
    case 304: return launch<K, CB, 3, 4>(a, st);
    case 312: return launch<K, CB, 3, 12>(a, st);
    case 208: return launch<K, CB, 2, 8>(a, st);
    case 308: return launch<K, CB, 3, 8>(a, st);
    default: return launch<K, CB, 4, 8>(a, st);
  }
}
}  // namespace gmid

// Tile choice: rows rb and token blocks nb (tokens spread evenly over the n_tt token tiles) with the
// least estimated time: a launch, and per round of workgroups (one per compute unit, a started round counts
// whole) a tile's start and end, its stores (twice as long where d_out is not a multiple of four) and, for
// 4096 inputs, dequantization per plane and 16 rows (8- and 4-bit codes) and X and the products per token block
// (longer where the rows of X don't start on whole lines). Fitted per shape to 3500 layers and token
// counts (d_out 200 .. 14000, d_in 200 .. 12000, 17 to 3000 tokens, both code widths, inputs and outputs
// rotated): 10 % are measured below 0.9 or above 1.15 of the estimate.
struct MidTile { int rb, nb_max, nb, n_tt; double us; };
static MidTile mid_tile(const Layer& L, int k, int n, int rb = 0, int nb_max = 0) {   // rb > 0: that shape only
  static const struct { int rb, nb; double launch, start, store, plane8, plane4, block, ragged; } shapes[9] = {
      {1, 2, 1.68, 2.63, 0.28, 0.61, 0.43, 1.05, 0.15}, {1, 4, 1.85, 3.10, 0.18, 0.62, 0.43, 1.12, 0.20},
      {2, 2, 1.59, 3.05, 0.16, 0.72, 0.55, 0.83, 0.11}, {2, 4, 1.50, 3.54, 0.15, 0.56, 0.45, 0.97, 0.17},
      {2, 8, 1.30, 4.65, 0.15, 0.67, 0.51, 0.92, 0.24}, {3, 4, 1.50, 4.03, 0.15, 0.77, 0.63, 0.82, 0.06},
      {3, 8, 1.61, 4.77, 0.11, 0.66, 0.57, 1.43, 0.10}, {3, 12, 1.75, 5.97, 0.10, 0.69, 0.59, 1.47, 0.13},
      {4, 8, 1.63, 5.19, 0.10, 0.67, 0.58, 1.54, 0.09}};
  const int ncu = L.n_cu > 0 ? L.n_cu : 256, blocks = (n + 15) / 16, odd = (L.d.d_out & 3) ? 2 : 1;
  const double len = L.d.d_in / 4096.0;
  MidTile best{};
  for (const auto& s : shapes) {
    if (rb > 0 && (s.rb != rb || s.nb != nb_max)) continue;
    const int tt = (blocks + s.nb - 1) / s.nb, b = (blocks + tt - 1) / tt;
    const long long wgs = (long long)((L.d.d_out + 16 * s.rb - 1) / (16 * s.rb)) * tt;
    const double plane = L.d.code_bits == 4 ? s.plane4 : s.plane8, block = s.block + (L.d.d_in % 64 ? s.ragged : 0.0);
    const double us = s.launch + (double)((wgs + ncu - 1) / ncu) *
                                     (s.start + s.store * b * s.rb * odd + len * (plane * s.rb * k + block * b));
    if (best.rb == 0 || us < best.us) best = {s.rb, s.nb, b, tt, us};
  }
  return best;
}

double gemm_mid_us(const Layer& L, int k, int n_tokens) {
  if (k > 4 || L.d.code_bits == 16 || L.d.d_in > (1 << 20)) return -1.0;
  return mid_tile(L, k, n_tokens).us;
}

hipError_t launch_gemm_mid(const Layer& L, int k, const void* X, int n_tokens, void* Y, aqmb_dtype y_dtype, int rb,
                           int nb_max, hipStream_t st) {
  const MidTile tile = mid_tile(L, k, n_tokens, rb, nb_max);
  if (tile.rb == 0) return hipErrorInvalidValue;
  gmid::Args a{};
  a.codes = L.codes;
  a.codebooks = L.codebooks;
  a.scales = L.scales;
  a.X = (const uint16_t*)X;
  a.Y = Y;
  a.zero_page = L.zero_page();
  a.plane_bytes = L.plane_bytes;
  a.d_out = L.d.d_out;
  a.d_in = L.d.d_in;
  a.G = L.G;
  a.n = n_tokens;
  a.y_dtype = (int)y_dtype;
  rb = tile.rb;
  nb_max = tile.nb_max;
  a.nb = tile.nb;
  a.n_tt = tile.n_tt;
  if (L.d.code_bits == 4) switch (k) {
    case 1: return gmid::launch_shape<1, 4>(a, rb, nb_max, st);
    case 2: return gmid::launch_shape<2, 4>(a, rb, nb_max, st);
    case 3: return gmid::launch_shape<3, 4>(a, rb, nb_max, st);
    default: return gmid::launch_shape<4, 4>(a, rb, nb_max, st);
  }
  switch (k) {
    case 1: return gmid::launch_shape<1, 8>(a, rb, nb_max, st);
    case 2: return gmid::launch_shape<2, 8>(a, rb, nb_max, st);
    case 3: return gmid::launch_shape<3, 8>(a, rb, nb_max, st);
    default: return gmid::launch_shape<4, 8>(a, rb, nb_max, st);
  }
}

}  // namespace aqmb
