// Kernel launchers (defined in the .hip files). Arguments are already validated.
#pragma once
#include <hip/hip_runtime.h>

#include "layer.h"

namespace aqmb {

// Re-tile n_planes plane-major code planes [n_planes][d_out][G] into out (n_planes tiled planes);
// for 4-bit codes a value above 15 sets *bad (device int).
hipError_t launch_retile(const Layer& L, const void* codes_plane_major, int n_planes, unsigned char* out, int* bad,
                         hipStream_t st);
hipError_t launch_dequant(const Layer& L, int k, void* W, aqmb_dtype w_dtype, hipStream_t st);
// Direct-gather GEMV of a layer with 8-bit codes; it serves the call when gemv_cw_fits.
bool gemv_cw_fits(const Layer& L, int k, int batch, aqmb_dtype x_dtype);
hipError_t launch_gemv_cw(const Layer& L, int k, const void* x, aqmb_dtype x_dtype, int batch, void* y,
                          aqmb_dtype y_dtype, hipStream_t st);
// Decode GEMV of a layer with 16-bit codes (codewords gathered through L2), any k, batch and row.
hipError_t launch_gemv_b16(const Layer& L, int k, const void* x, aqmb_dtype x_dtype, int batch, void* y,
                           aqmb_dtype y_dtype, hipStream_t st);
// Lookup-table GEMV (8-bit codes): split-K partial sums in `scratch` (gemv_lut_scratch_bytes bytes,
// owned by the caller for the duration of the launch on st).
size_t gemv_lut_scratch_bytes(const Layer& L, int batch);
hipError_t launch_gemv_lut(const Layer& L, int k, const void* x, aqmb_dtype x_dtype, int batch, void* y,
                           aqmb_dtype y_dtype, float* scratch, hipStream_t st);
// Decode GEMV of a layer with 8- or 4-bit codes on the matrix cores (batch 1..16).
hipError_t launch_gemv_mma(const Layer& L, int k, const void* x, aqmb_dtype x_dtype, int batch, void* y,
                           aqmb_dtype y_dtype, hipStream_t st);
// The same for n layers with the same d_in, code width and device, in one launch (results equal to
// launch_gemv_mma's for each layer); n <= AQMB_MAX_MULTI.
hipError_t launch_gemv_mma_multi(const Layer* const* Ls, int n, int k, const void* x, aqmb_dtype x_dtype, int batch,
                                 void* const* ys, aqmb_dtype y_dtype, hipStream_t st);
bool gemv_mma_multi_fits(const Layer* const* Ls, int n, int k, int batch, aqmb_dtype x_dtype);
// Decode GEMV of a layer with 4-bit codes (16-codeword codebooks).
hipError_t launch_gemv_b4(const Layer& L, int k, const void* x, aqmb_dtype x_dtype, int batch, void* y,
                          aqmb_dtype y_dtype, hipStream_t st);
// Several layers with the same d_in and device, already validated; n <= AQMB_MAX_MULTI.
hipError_t launch_gemv_multi(const Layer* const* Ls, int n, int k, const void* x, aqmb_dtype x_dtype, int batch,
                             void* const* ys, aqmb_dtype y_dtype, hipStream_t st);
// All prefix distortions D[0..M-1] of the layer against fp16 W [d_out][d_in] and fp16 inputs
// X [n][d_in]; the per-workgroup sums go to `scratch` (distortion_scratch_bytes bytes).
hipError_t launch_distortion(const Layer& L, const void* W, const void* X, int n, double* D, double* scratch,
                             hipStream_t st);
size_t distortion_scratch_bytes();
// The device address of the distortion's file-scope scratch array on `device` (which must be
// current), looked up on the first call per device; *bytes is its size.
hipError_t distortion_static_scratch(int device, double** out, size_t* bytes);
// Beam search of codes for every group of W [d_out][d_in] fp16 over codebooks 0..k-1 (8-bit).
hipError_t launch_beam_search(const aqmb_desc& d, int k, int beam_width, const void* W, const uint16_t* codebooks,
                              const uint16_t* scales, unsigned char* codes, float* errors, hipStream_t st);
// The same search for the data-aware objective d^T H_jj d (H: [G][8][8] fp32 symmetric blocks).
hipError_t launch_beam_search_weighted(const aqmb_desc& d, int k, int beam_width, const void* W,
                                       const uint16_t* codebooks, const uint16_t* scales, const float* H,
                                       unsigned char* codes, float* errors, hipStream_t st);
// Both searches for 8-bit codes and beams of at most 8 (H null: the plain objective), the matrix cores
// as a filter; the same codes and errors bit for bit.
hipError_t launch_beam_mma(const aqmb_desc& d, int k, int beam_width, const void* W, const uint16_t* codebooks,
                           const uint16_t* scales, const float* H, unsigned char* codes, float* errors, hipStream_t st);
// Prefill GEMM tiled for small token counts (same arithmetic as launch_gemm), and its estimated time, k <= 4.
double gemm_small_us(const Layer& L, int k, int n_tokens);
hipError_t launch_gemm_small(const Layer& L, int k, const void* X, int n_tokens, void* Y, aqmb_dtype y_dtype,
                             hipStream_t st);
// Addresses in a token tile of the split-input GEMM: tokens t0 .. t0 + 16 nb - 1 of n, 32-bit byte
// offsets from the tile's first token. The tile's last row is taken before it is multiplied: n - t0 rows
// of X may span more than 2^32 bytes, 16 nb rows of at most 2^21 bytes do not.
__host__ __device__ inline uint32_t gemm_mid_last_row(int n, int t0, int nb) {
  const int left = n - 1 - t0, tile = 16 * nb - 1;
  return (uint32_t)(left < tile ? left : tile);
}
__host__ __device__ inline uint32_t gemm_mid_x_offset(uint32_t row, uint32_t row_bytes, uint32_t piece) {
  return row * row_bytes + piece * 16;
}
// Prefill GEMM for tens to hundreds of tokens, k <= 4 (same arithmetic).
// gemm_mid_us: its estimated time (-1 where it does not serve the call).
double gemm_mid_us(const Layer& L, int k, int n_tokens);
// rb, nb_max: weight rows / 16 and token blocks of the tile (0, 0: the rule's choice; a pair that is not
// one of its nine shapes is hipErrorInvalidValue).
hipError_t launch_gemm_mid(const Layer& L, int k, const void* X, int n_tokens, void* Y, aqmb_dtype y_dtype, int rb,
                           int nb_max, hipStream_t st);
// Large-tile prefill GEMM; tile: -1 = chosen by the number of workgroup rounds, 0 = 256 x 128,
// 1 = 128 x 128, 2 = 128 x 64 (tokens x weight rows).
hipError_t launch_gemm(const Layer& L, int k, const void* X, int n_tokens, void* Y, aqmb_dtype y_dtype, int tile,
                       hipStream_t st);
// Estimated time of launch_gemm's choice of tile, k <= 4.
double gemm_large_us(const Layer& L, int k, int n_tokens);
// Two-pass prefill GEMM (bit-identical to the 256 x 128 tiling): workspace bytes (0 where it does
// not apply) and the launch (workspace of at least that many bytes, 256-byte aligned).
size_t gemm_two_pass_bytes(const Layer& L, int k, int n_tokens);
bool gemm_dense256(const Layer& L, int n_tokens);            // its dense pass takes 256 x 256 tiles
hipError_t launch_gemm_two_pass(const Layer& L, int k, const void* X, int n_tokens, void* Y, aqmb_dtype y_dtype,
                                void* workspace, hipStream_t st);

}  // namespace aqmb
