// Code re-tiling (layer creation) and the bit-exact dequantization kernel.
#include <algorithm>

#include "device.h"
#include "launch.h"

namespace aqmb {

// [M][d_out][G] plane-major codes -> [M][S][d_out][16 bytes]. CB = code bits: 16-bit codes are
// 2 bytes each, 8-bit and 4-bit codes 1 byte each in the input; a slice holds J = 128 / CB
// consecutive groups of one row, 4-bit codes packed two to a byte (group 2b in the low nibble of
// byte b, group 2b + 1 in the high nibble). A 4-bit code above 15 sets *bad (the layer is refused).
template <int CB>
__global__ __launch_bounds__(256) void retile_kernel(const unsigned char* __restrict__ in, unsigned char* __restrict__ out,
                                                     int M, int d_out, int G, int S, int* bad) {
  constexpr int J = 128 / CB, CS = CB == 16 ? 2 : 1;
  const size_t total = (size_t)M * S * d_out;
  for (size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x; q < total; q += (size_t)gridDim.x * blockDim.x) {
    const int i = (int)(q % d_out);
    const size_t ms = q / d_out;
    const int s = (int)(ms % S), m = (int)(ms / S);
    unsigned char chunk[16];
    if constexpr (CB == 4) {
      unsigned high = 0;
#pragma unroll
      for (int b = 0; b < 16; ++b) {
        const int j0 = s * J + 2 * b, j1 = j0 + 1;
        const unsigned c0 = j0 < G ? in[((size_t)m * d_out + i) * G + j0] : 0u;
        const unsigned c1 = j1 < G ? in[((size_t)m * d_out + i) * G + j1] : 0u;
        high |= (c0 | c1) >> 4;
        chunk[b] = (unsigned char)((c0 & 15u) | ((c1 & 15u) << 4));
      }
      if (high) *bad = 1;
    } else {
#pragma unroll
      for (int jj = 0; jj < J; ++jj) {
        const int j = s * J + jj;
#pragma unroll
        for (int b = 0; b < CS; ++b)
          chunk[jj * CS + b] = j < G ? in[(((size_t)m * d_out + i) * G + j) * CS + b] : (unsigned char)0;
      }
    }
    uint4 v;
    __builtin_memcpy(&v, chunk, 16);
    *(uint4*)(out + q * 16) = v;
  }
}

hipError_t launch_retile(const Layer& L, const void* codes, int n_planes, unsigned char* out, int* bad,
                         hipStream_t st) {
  const size_t total = (size_t)n_planes * L.S * L.d.d_out;
  const unsigned grid = (unsigned)((total + 255) / 256 < 65536 ? (total + 255) / 256 : 65536);
  const auto* in = (const unsigned char*)codes;
  if (L.d.code_bits == 8)
    retile_kernel<8><<<grid, 256, 0, st>>>(in, out, n_planes, L.d.d_out, L.G, L.S, bad);
  else if (L.d.code_bits == 4)
    retile_kernel<4><<<grid, 256, 0, st>>>(in, out, n_planes, L.d.d_out, L.G, L.S, bad);
  else
    retile_kernel<16><<<grid, 256, 0, st>>>(in, out, n_planes, L.d.d_out, L.G, L.S, bad);
  return hipGetLastError();
}

// The stated evaluation order for W_k: binary32 left fold over planes, one binary32
// multiply by the row scale, one rounding to the output format. Contraction into a
// fused multiply-add is off so every step rounds on its own.
#pragma clang fp contract(off)

// The output is written once and not read back by this kernel: streaming (nontemporal) stores.
__device__ __forceinline__ void store_stream16(void* p, uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  const u32x4_t v = {a, b, c, d};
  __builtin_nontemporal_store(v, (u32x4_t*)p);
}

template <int OUT>
__device__ __forceinline__ void store_group(void* W, size_t elem, const float (&w)[8]) {
  if constexpr (OUT == AQMB_F32) {
    float* p = (float*)W + elem;
    store_stream16(p, __float_as_uint(w[0]), __float_as_uint(w[1]), __float_as_uint(w[2]), __float_as_uint(w[3]));
    store_stream16(p + 4, __float_as_uint(w[4]), __float_as_uint(w[5]), __float_as_uint(w[6]), __float_as_uint(w[7]));
  } else if constexpr (OUT == AQMB_F16) {
    store_stream16((uint16_t*)W + elem, pack_f16x2(w[0], w[1]), pack_f16x2(w[2], w[3]),
                   pack_f16x2(w[4], w[5]), pack_f16x2(w[6], w[7]));
  } else {
    store_stream16((uint16_t*)W + elem, pack_bf16x2(w[0], w[1]), pack_bf16x2(w[2], w[3]),
                   pack_bf16x2(w[4], w[5]), pack_bf16x2(w[6], w[7]));
  }
}

// acc = the first codeword (exact in binary32), or acc + the codeword, one rounding per element
__device__ __forceinline__ void fold_codeword(float (&acc)[8], uint4 cw, bool first) {
  if (first) {
    acc[0] = f16lo(cw.x); acc[1] = f16hi(cw.x); acc[2] = f16lo(cw.y); acc[3] = f16hi(cw.y);
    acc[4] = f16lo(cw.z); acc[5] = f16hi(cw.z); acc[6] = f16lo(cw.w); acc[7] = f16hi(cw.w);
  } else {
    acc[0] = add_f16_lo(cw.x, acc[0]); acc[1] = add_f16_hi(cw.x, acc[1]);
    acc[2] = add_f16_lo(cw.y, acc[2]); acc[3] = add_f16_hi(cw.y, acc[3]);
    acc[4] = add_f16_lo(cw.z, acc[4]); acc[5] = add_f16_hi(cw.z, acc[5]);
    acc[6] = add_f16_lo(cw.w, acc[6]); acc[7] = add_f16_hi(cw.w, acc[7]);
  }
}

// c0 + c1 for the fp16 values in the low (or high) halves of a and b, rounded once to binary32:
// the first two steps of the fold in one instruction (an fma with 1.0 and both sources fp16).
__device__ __forceinline__ float add2_f16_lo(uint32_t a, uint32_t b) {
  float d;
  asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel_hi:[1,0,1]" : "=v"(d) : "v"(b), "v"(a));
  return d;
}
__device__ __forceinline__ float add2_f16_hi(uint32_t a, uint32_t b) {
  float d;
  asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel:[1,0,1] op_sel_hi:[1,0,1]" : "=v"(d) : "v"(b), "v"(a));
  return d;
}

// acc = (binary32) c0 + c1, elementwise
__device__ __forceinline__ void fold_first_two(float (&acc)[8], uint4 c0, uint4 c1) {
  acc[0] = add2_f16_lo(c0.x, c1.x); acc[1] = add2_f16_hi(c0.x, c1.x);
  acc[2] = add2_f16_lo(c0.y, c1.y); acc[3] = add2_f16_hi(c0.y, c1.y);
  acc[4] = add2_f16_lo(c0.z, c1.z); acc[5] = add2_f16_hi(c0.z, c1.z);
  acc[6] = add2_f16_lo(c0.w, c1.w); acc[7] = add2_f16_hi(c0.w, c1.w);
}

// 16 times byte j of w (the LDS byte offset of that code's codeword), one instruction; j must be
// a constant after unrolling.
__device__ __forceinline__ uint32_t code_x16(uint32_t w, int j) {
  uint32_t d;
  switch (j) {
    case 0: asm("v_lshlrev_b32_sdwa %0, 4, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_0" : "=v"(d) : "v"(w)); break;
    case 1: asm("v_lshlrev_b32_sdwa %0, 4, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_1" : "=v"(d) : "v"(w)); break;
    case 2: asm("v_lshlrev_b32_sdwa %0, 4, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_2" : "=v"(d) : "v"(w)); break;
    default: asm("v_lshlrev_b32_sdwa %0, 4, %1 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_3" : "=v"(d) : "v"(w)); break;
  }
  return d;
}

// Small layers: one thread per group (J = 128 / CB lanes for the groups of a (slice, row) pair), all of them
// running at once. Bound: the latency of one chain - codebooks and code word in flight together, gather,
// fold, store - against which the pieces of rows that a store instruction writes here do not count. 512 x 512,
// k = 1 / 4, us (an empty kernel of that size: 2.3): 8-bit codes to bf16 3.8 / 4.8 -> 2.3 / 2.4, 4-bit codes
// 4.7 / 5.5 -> 2.3 / 2.4; 16-bit codes, 2048 x 2048 to bf16, k = 1 / 2, 7.0 / 8.3 -> 5.1 / 7.0.
template <int OUT, int CB, int K>
__global__ __launch_bounds__(256) void dequant_small_kernel(const unsigned char* codes, const uint16_t* codebooks,
                                                            const uint16_t* scales, void* W, int d_out, int d_in, int G,
                                                            uint32_t nslot, size_t plane_bytes) {
  constexpr int NCW = 1 << CB, J = 128 / CB, PER_WORD = 32 / CB;
  __shared__ uint4 cbs[CB <= 8 ? K * NCW : 1];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if constexpr (CB == 8) {
#pragma unroll
    for (int i = 0; i < K; ++i) load_lds16((const uint4*)codebooks + i * 256 + tid, lds_addr(cbs + i * 256 + wave * 64));
  } else if constexpr (CB == 4) {
    if (tid < K * NCW) cbs[tid] = ((const uint4*)codebooks)[tid];
  }
  uint32_t slot = blockIdx.x * 256 + tid;
  const bool live = slot < nslot;
  slot = live ? slot : nslot - 1;                      // past the end: the last slot again, not stored
  const uint32_t pair = slot / J, jj = slot % J, slice = pair / (uint32_t)d_out;
  const int row = (int)(pair - slice * (uint32_t)d_out), grp = (int)(slice * J + jj);
  const float scale = f16_to_f32(scales[row]);
  uint32_t w[K];
#pragma unroll
  for (int m = 0; m < K; ++m) w[m] = *(const uint32_t*)(codes + m * plane_bytes + (size_t)pair * 16 + jj / PER_WORD * 4);
  if constexpr (CB <= 8) {
    wait_vmcnt<0>();
    __syncthreads();
  }
  if (!live || grp >= G) return;
  float acc[8];
#pragma unroll
  for (int m = 0; m < K; ++m) {
    const uint32_t code = (w[m] >> (CB * (jj % PER_WORD))) & (NCW - 1);
    fold_codeword(acc, CB <= 8 ? cbs[m * NCW + code] : ((const uint4*)codebooks)[((size_t)m << 16) + code], m == 0);
  }
  float v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    v[e] = acc[e] * scale;
    asm volatile("" : "+v"(v[e]));                     // keep the binary32 product: no fused multiply and conversion
  }
  store_group<OUT>(W, (size_t)row * d_in + (size_t)grp * 8, v);
}

// 8-bit codes to 16 bits, middle and very large layers (see launch_dequant_k): tiles of RT rows x GT groups
// (RT GT = 2048 or 4096 groups, 32 or 64 KiB of output), 512 threads.
// Thread t takes row t % RT of the tile and P = RT GT / 512 consecutive groups of it (part (t / RT) of the
// tile's GT / 16 slices): one P-byte code load per plane brings them, which it folds into the tile in LDS,
// row-major, its 16-byte chunks XOR-swizzled by row so that both the column-wise writes and the row-wise
// reads hit every bank group. Then the waves write the tile row by row, 1 KiB contiguous per store
// instruction and P of them back to back, which HBM takes faster than the steady trickle of
// dequant_kernel. Tiles are numbered column tiles fastest, so the tiles in flight together cover whole rows
// of the output. A workgroup walks its tiles with the grid's stride; the code words of its next tile are
// requested before the current one is folded.
namespace dq {
constexpr int kThreads = 512, kWaves = kThreads / 64;
}

// LDS writes of this wave complete, then a workgroup barrier (global loads stay in flight).
__device__ __forceinline__ void dq_lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);                  // lgkmcnt(0); vmcnt and expcnt at their maxima
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

template <int OUT, int K, int RT, int GT>
__global__ __launch_bounds__(dq::kThreads) void dequant8_tile_kernel(const unsigned char* codes, const uint16_t* codebooks,
                                                                    const uint16_t* scales, void* W, int d_out, int d_in,
                                                                    int G, int S, size_t plane_bytes) {
  static_assert(OUT == AQMB_F16 || OUT == AQMB_BF16, "16-bit outputs");
  static_assert(RT * GT == 4096 || RT * GT == 2048, "tile size");
  static_assert(GT >= 64 && (GT & (GT - 1)) == 0 && RT <= 64, "swizzle range");
  using namespace dq;
  constexpr int P = RT * GT / kThreads, kParts = 16 / P, ST = GT / 16, CP = GT / 64;
  // static LDS, codebooks first: their addresses fit the reads' offset field
  __shared__ struct {
    uint4 cb[K * 256];                                 // [K][256] codewords
    uint4 tile[RT * GT];                               // [RT rows][GT chunks of 16 bytes], swizzled
  } sm;
  uint4* cb8 = sm.cb;
  uint4* tile = sm.tile;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  for (int q = tid; q < K * 256; q += kThreads) cb8[q] = ((const uint4*)codebooks)[q];
  const int n_ct = (S + ST - 1) / ST, n_tiles = n_ct * ((d_out + RT - 1) / RT);
  const int rl = tid % RT, q = tid / RT, sl_t = q / kParts, part = q % kParts;   // row, slice, part of the slice
  uint2 c[K];
  uint32_t sc = 0;
  // code words (P bytes per plane) and row scale of tile t for this thread; tiles past the end
  // reload the last one, rows and slices past the layer reload its last row and slice (never stored)
  auto load = [&](int t) {
    const int tc = t < n_tiles ? t : n_tiles - 1;
    int row = (tc / n_ct) * RT + rl, sl = (tc % n_ct) * ST + sl_t;
    row = row < d_out ? row : d_out - 1;
    sl = sl < S ? sl : S - 1;
    sc = scales[row];
    const unsigned char* p = codes + ((size_t)sl * d_out + row) * 16 + part * P;
#pragma unroll
    for (int m = 0; m < K; ++m) {
      if constexpr (P == 8) c[m] = load_stream8(p + m * plane_bytes);
      else c[m] = make_uint2(__builtin_nontemporal_load((const uint32_t*)(p + m * plane_bytes)), 0u);
    }
  };
  int t = blockIdx.x;
  load(t);
  __syncthreads();
  for (; t < n_tiles; t += gridDim.x) {
    const int r0 = (t / n_ct) * RT, g0 = (t % n_ct) * GT;
    const float scale = f16_to_f32((uint16_t)sc);
    uint2 w[K];
#pragma unroll
    for (int m = 0; m < K; ++m) w[m] = c[m];
    load(t + gridDim.x);
#pragma unroll
    for (int jj = 0; jj < P; ++jj) {
      uint4 cw[K];
#pragma unroll
      for (int m = 0; m < K; ++m)
        cw[m] = *(const uint4*)((const char*)(cb8 + m * 256) + code_x16(jj < 4 ? w[m].x : w[m].y, jj & 3));
      float acc[8];
      if constexpr (K == 1) fold_codeword(acc, cw[0], true);
      else fold_first_two(acc, cw[0], cw[1]);
#pragma unroll
      for (int m = 2; m < K; ++m) fold_codeword(acc, cw[m], false);
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        v[e] = acc[e] * scale;
        asm volatile("" : "+v"(v[e]));  // keep the binary32 product: no fused multiply and conversion
      }
      const uint4 o = OUT == AQMB_F16
                          ? make_uint4(pack_f16x2(v[0], v[1]), pack_f16x2(v[2], v[3]), pack_f16x2(v[4], v[5]), pack_f16x2(v[6], v[7]))
                          : make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]),
                                       pack_bf16x2(v[6], v[7]));
      const int chunk = sl_t * 16 + part * P + jj;
      tile[rl * GT + (chunk ^ rl)] = o;
    }
    dq_lds_barrier();
    // P stores per wave: store j = wave P + i writes chunk part j % CP of tile row j / CP
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const int j = wave * P + i, r = j / CP, ch = (j % CP) * 64 + lane, row = r0 + r, grp = g0 + ch;
      const uint4 o = tile[r * GT + (ch ^ r)];
      if (row < d_out && grp < G) store_stream16((uint16_t*)W + (size_t)row * d_in + (size_t)grp * 8, o.x, o.y, o.z, o.w);
    }
    dq_lds_barrier();                                   // the tile is read before the next one is written
  }
}

// Dequantization, every code width and output type. Bound: the stores of W (the codes are 1/16 to 1/4 of
// them), and for 65536-entry codebooks the gathers of codewords through the L2.
// A wave takes units of R rows x 64 groups. It loads the unit's code slices (per plane one load, R rows x
// 16 bytes of each slice), turns them through its own LDS so that lane l finds the code of group l (fp32
// output: of group l / 2, the lane making its half of the group), gathers and folds the codewords and
// stores them: every store instruction writes 1 KiB of one row (64 rows x 256-byte pieces, which a lane
// per group in code order gives, cost 2.5 x as much at fp32), and no wave waits for another after the
// codebooks are staged. Units are numbered along the rows, so that the waves of a workgroup write whole
// rows between them; the next unit's codes are requested before the current unit is folded. 16- and
// 256-entry codebooks are staged in LDS, 65536-entry ones are read through the caches.
// Measured on the 4096 x 11008 layer, us (fill of the same output: 15.0 at 16 bits, 28.2 at 32), before:
// a kernel with a workgroup-wide output tile for 8-bit codes to 16 bits, a thread per group for the rest:
//   8-bit codes   bf16 k = 1..4  20.8 22.5 24.2 26.6 -> 18.1 18.8 18.8 21.0   fp32  84 79 75 73 -> 35 36 37 39
//   4-bit codes   bf16 k = 1..4  23.8                -> 18.1 18.3 18.8 19.0   fp32  84          -> 35 36 36 37
//   16-bit codes  (bf16, and fp32 at k = 2: thread per group)                fp32 k = 1  66 -> 41
template <int CB, int K, int R, int NW> constexpr size_t dequant_lds() {
  return (CB <= 8 ? (size_t)K * (1 << CB) * 16 : 0) + (size_t)NW * K * R * 8 * CB;
}

template <int OUT, int CB, int K, int R, int NW>
__global__ __launch_bounds__(64 * NW) void dequant_kernel(const unsigned char* codes, const uint16_t* codebooks,
                                                          const uint16_t* scales, void* W, int d_out, int d_in, int G, int S,
                                                          size_t plane_bytes, int n_units, int n_ct) {
  constexpr int NCW = 1 << CB, NSL = CB / 2, kRowB = 8 * CB;   // slices, code bytes of a unit's row
  constexpr bool F32 = OUT == AQMB_F32;
  extern __shared__ uint4 dequant_smem[];
  uint4* cbs = dequant_smem;                           // [K][NCW] codewords (CB <= 8)
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  unsigned char* buf = (unsigned char*)(dequant_smem + (CB <= 8 ? K * NCW : 0)) + wave * K * R * kRowB;
  const int lr = lane % R, ls = lane / R;              // row and slice this lane loads (ls < NSL)
  uint4 c[K];
  uint32_t sc = 0;
  auto load = [&](int u) {                             // units past the end reload the last one
    u = u < n_units ? u : n_units - 1;
    int row = (u / n_ct) * R + lr, sl = (u % n_ct) * NSL + ls;
    row = row < d_out ? row : d_out - 1;
    sl = sl < S ? sl : S - 1;
    sc = scales[row];
    if (ls < NSL) {
#pragma unroll
      for (int m = 0; m < K; ++m) c[m] = load_stream16(codes + m * plane_bytes + ((size_t)sl * d_out + row) * 16);
    }
  };
  int u = blockIdx.x * NW + wave;
  if constexpr (CB == 8) {
#pragma unroll
    for (int q = 0; q < K * NCW / 64; q += NW)
      if (q + wave < K * NCW / 64) load_lds16((const uint4*)codebooks + (q + wave) * 64 + lane, lds_addr(cbs + (q + wave) * 64));
  } else if constexpr (CB == 4) {
    if (tid < K * NCW) cbs[tid] = ((const uint4*)codebooks)[tid];
  }
  load(u);
  if constexpr (CB <= 8) {
    wait_vmcnt<0>();
    __syncthreads();
  }
  const int gl = F32 ? lane >> 1 : lane;               // this lane's group of a row (fp32: of each half unit)
  for (; u < n_units; u += gridDim.x * NW) {
    const int r0 = (u / n_ct) * R, g0 = (u % n_ct) * 64;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the previous unit's code reads precede these writes
    __builtin_amdgcn_wave_barrier();
    if (ls < NSL) {
#pragma unroll
      for (int m = 0; m < K; ++m) *(uint4*)(buf + (m * R + lr) * kRowB + ls * 16) = c[m];
    }
    const uint32_t scales8 = sc;                       // lane r: the scale of row r0 + r
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    load(u + gridDim.x * NW);
    auto get = [&](int r, int m, int g) -> uint32_t {
      const unsigned char* p = buf + (m * R + r) * kRowB;
      if constexpr (CB == 16) return ((const uint16_t*)p)[g];
      else if constexpr (CB == 8) return p[g];
      else return (p[g >> 1] >> (4 * (g & 1))) & 15u;
    };
#pragma unroll
    for (int r = 0; r < R; ++r) {
      // 16-bit codes: the branch keeps the gathers of one row together (33.5 us, against 35.2 without it)
      if (CB == 16 && r0 + r >= d_out) break;
      const float scale = f16_to_f32(__builtin_amdgcn_readlane(scales8, r));
#pragma unroll
      for (int h = 0; h < (F32 ? 2 : 1); ++h) {
        const int g = h * 32 + gl;
        uint4 cw[K];
#pragma unroll
        for (int m = 0; m < K; ++m) {
          const uint32_t code = get(r, m, g);
          const uint4* src = CB <= 8 ? cbs + ((uint32_t)(m * NCW) + code)
                                     : (const uint4*)codebooks + (((size_t)m << 16) + code);
          if constexpr (F32) {
            const uint2 v = ((const uint2*)src)[lane & 1];
            cw[m] = make_uint4(v.x, v.y, 0u, 0u);
          } else {
            cw[m] = *src;
          }
        }
        float acc[8];
        if constexpr (K == 1) fold_codeword(acc, cw[0], true);
        else fold_first_two(acc, cw[0], cw[K > 1 ? 1 : 0]);
#pragma unroll
        for (int m = 2; m < K; ++m) fold_codeword(acc, cw[m], false);
        float v[8];
#pragma unroll
        for (int e = 0; e < (F32 ? 4 : 8); ++e) {
          v[e] = acc[e] * scale;
          asm volatile("" : "+v"(v[e]));               // keep the binary32 product: no fused multiply and conversion
        }
        if (r0 + r >= d_out || g0 + g >= G) continue;
        const size_t o = (size_t)(r0 + r) * d_in + (size_t)(g0 + g) * 8;
        if constexpr (F32)
          store_stream16((float*)W + o + 4 * (lane & 1), __float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]),
                         __float_as_uint(v[3]));
        else
          store_group<OUT>(W, o, v);
      }
    }
  }
}

// Which kernel. Times in us, 256 compute units; "cold": codes and outputs rotated through 0.7 GB.
// - A thread per group: 16-bit outputs while all threads run at once (2048 per compute unit; 2048 x 2048, 8-bit
//   codes, k = 1 / 4, cold: 3.4 / 4.0 against 4.5 / 5.2 with output tiles), fp32 up to 640 threads per unit
//   (1000 x 1032: 3.8 / 4.0 against 3.8 / 4.3 on wave units; 333 x 8200: 6.0 / 6.3 against 4.9 / 5.7).
//   65536-entry codebooks: always but for fp32 at k = 1 past 1536 threads per unit, where the gathers are
//   few enough for the stores to count (cold, against wave units: 11008 x 4096 to bf16, k = 1 / 2, 29.5 / 52.4
//   against 32.5 / 54.8, to fp32 49.7 / 63.1 against 41.2 / 70.7).
// - dequant8_tile_kernel, 8-bit codes to 16 bits: one tile per workgroup while a layer has at most two 64 KiB
//   tiles per compute unit (cold, against wave units: 4096 x 4096, k = 1..4, 8.6 8.7 9.0 9.7 against 10.2 9.6 10.3
//   10.7, whose 4-row units read half lines), and 32 x 64 tiles once codes and output pass 148 MiB (14336 x
//   4096, k = 6 / 8, 154 and 168 MiB: 34 / 37 against 37 / 41, k = 4, 140 MiB: 32 against 29; 28672 x 8192: 91 / 112
//   at k = 1 / 4 against 100 / 122). From k = 3 on also where the wave units leave compute units idle (each wave one
//   unit, workgroups filling less than 0.85 of their last round: 2116 x 8192, k = 4, cold, 14.0 against 16.8, 5120 x
//   4096 14.1 against 16.4) or rows don't start on whole 128-byte lines and waves walk several units (11386 x 4912, k = 3,
//   31.1 against 33.9; 5063 x 11272, k = 4, 37.5 against 40.5). Of 210 ragged layers at k = 3 and 4, units were more
//   than 3 % slower than tiles on 86, with this rule on 12; mean 1.003 -> 0.985 of the tiles' time. At k >= 5 always
//   (150 ragged layers: units 2.3 % slower on average, more than 3 % on 47).
// - dequant_kernel for the rest, with at most as many workgroups as run at once, each wave walking its units
//   with the grid's stride. Units of 8 rows (whole lines of codes), 8-wave workgroups where every wave gets a
//   unit (8 per compute unit at k >= 3, 16 at k <= 2, where a unit is soon done), else 4-wave ones (4096 x 4096 to
//   fp32, k = 1, cold: 16.6 against 19.0 with 4 rows and 8 waves); 4 rows where 4-row units would give 8 to 12 waves
//   per compute unit (1500 x 3000) and 2 where fewer than 6 (1000 x 1032, k = 2: 3.3 against 3.6), so that no unit
//   of the card stands idle.
template <int OUT, int CB, int K>
static void launch_dequant_k(const Layer& L, void* W, hipStream_t st) {
  const int d_out = L.d.d_out, ncu = L.n_cu > 0 ? L.n_cu : 256, n_ct = (L.G + 63) / 64;
  const size_t nslot = (size_t)L.S * d_out * (128 / CB);
  const int resident = OUT != AQMB_F32 ? 2048 : CB == 16 ? 1536 : 640;
  const bool gathers = CB == 16 && (OUT != AQMB_F32 || K > 1) && nslot < ((size_t)1 << 30);
  if (nslot <= (size_t)resident * ncu || gathers) {
    dequant_small_kernel<OUT, CB, K><<<(unsigned)((nslot + 255) / 256), 256, 0, st>>>(
        L.codes, L.codebooks, L.scales, W, d_out, L.d.d_in, L.G, (uint32_t)nslot, L.plane_bytes);
    return;
  }
  if constexpr (CB == 8 && OUT != AQMB_F32) {
    auto n_tiles = [&](int rt, int gt) { return ((d_out + rt - 1) / rt) * ((L.S + gt / 16 - 1) / (gt / 16)); };
    auto tiles = [&](auto kern, int grid) {
      kern<<<(unsigned)std::min(grid, 65535), dq::kThreads, 0, st>>>(L.codes, L.codebooks, L.scales, W, d_out, L.d.d_in, L.G,
                                                                     L.S, L.plane_bytes);
    };
    if (nslot < ((size_t)1 << 30)) {
      if (n_tiles(64, 64) <= 2 * ncu) {                // one tile per workgroup, as wide as the rows allow
        if (L.G > 256) tiles(dequant8_tile_kernel<OUT, K, 8, 512>, n_tiles(8, 512));
        else if (L.G > 128) tiles(dequant8_tile_kernel<OUT, K, 16, 256>, n_tiles(16, 256));
        else if (L.G > 64) tiles(dequant8_tile_kernel<OUT, K, 32, 128>, n_tiles(32, 128));
        else tiles(dequant8_tile_kernel<OUT, K, 64, 64>, n_tiles(64, 64));
        return;
      }
      bool tile = K >= 5 || (size_t)d_out * L.d.d_in * 2 + K * L.plane_bytes > ((size_t)148 << 20);
      const int wgs = (n_ct * ((d_out + 7) / 8) + 7) / 8;  // workgroups of wave units, one unit a wave
      if (K >= 3 && wgs > ncu) {
        const int per_cu = std::min<int>(160 * 1024 / (int)dequant_lds<CB, K, 8, 8>(), 4);
        tile = tile || (wgs <= per_cu * ncu ? wgs < 0.85 * ncu * ((wgs + ncu - 1) / ncu) : L.d.d_in % 64 != 0);
      }
      if (tile) {
        tiles(dequant8_tile_kernel<OUT, K, 32, 64>, std::min(n_tiles(32, 64), 2 * ncu));
        return;
      }
    }
  }
  auto go = [&](auto kern, size_t lds, int rows, int nw) {
    const int n_units = n_ct * ((d_out + rows - 1) / rows);
    const int per_cu = std::min<int>(160 * 1024 / (int)lds, 32 / nw);
    const int grid = std::min((n_units + nw - 1) / nw, per_cu * ncu);
    kern<<<grid, 64 * nw, lds, st>>>(L.codes, L.codebooks, L.scales, W, d_out, L.d.d_in, L.G, L.S, L.plane_bytes, n_units,
                                     n_ct);
  };
  const size_t u8 = (size_t)n_ct * ((d_out + 7) / 8), u4 = (size_t)n_ct * ((d_out + 3) / 4), cus = ncu;
  if (u8 > (K <= 2 ? 16 : 8) * cus) {
    go(dequant_kernel<OUT, CB, K, 8, 8>, dequant_lds<CB, K, 8, 8>(), 8, 8);
  } else if (CB != 16 && u4 < 6 * cus) {
    go(dequant_kernel<OUT, CB, K, 2, 4>, dequant_lds<CB, K, 2, 4>(), 2, 4);
  } else if (CB != 16 && u4 > 8 * cus && u4 < 12 * cus) {
    go(dequant_kernel<OUT, CB, K, 4, 4>, dequant_lds<CB, K, 4, 4>(), 4, 4);
  } else {
    go(dequant_kernel<OUT, CB, K, 8, 4>, dequant_lds<CB, K, 8, 4>(), 8, 4);
  }
}

template <int OUT, int CB>
static void launch_dequant_cb(const Layer& L, int k, void* W, hipStream_t st) {
  switch (k) {
    case 1: launch_dequant_k<OUT, CB, 1>(L, W, st); break;
    case 2: launch_dequant_k<OUT, CB, 2>(L, W, st); break;
    case 3: launch_dequant_k<OUT, CB, 3>(L, W, st); break;
    case 4: launch_dequant_k<OUT, CB, 4>(L, W, st); break;
    case 5: launch_dequant_k<OUT, CB, 5>(L, W, st); break;
    case 6: launch_dequant_k<OUT, CB, 6>(L, W, st); break;
    case 7: launch_dequant_k<OUT, CB, 7>(L, W, st); break;
    
    default: launch_dequant_k<OUT, CB, 8>(L, W, st); break;
  }
}

template <int OUT>
static void launch_dequant_out(const Layer& L, int k, void* W, hipStream_t st) {
  if (L.d.code_bits == 8) launch_dequant_cb<OUT, 8>(L, k, W, st);
  else if (L.d.code_bits == 4) launch_dequant_cb<OUT, 4>(L, k, W, st);
  else launch_dequant_cb<OUT, 16>(L, k, W, st);
}

hipError_t launch_dequant(const Layer& L, int k, void* W, aqmb_dtype w_dtype, hipStream_t st) {
  if (w_dtype == AQMB_F32) launch_dequant_out<AQMB_F32>(L, k, W, st);
  else if (w_dtype == AQMB_F16) launch_dequant_out<AQMB_F16>(L, k, W, st);
  else launch_dequant_out<AQMB_BF16>(L, k, W, st);
  return hipGetLastError();
}

}  // namespace aqmb
