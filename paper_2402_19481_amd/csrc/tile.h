// Shared by the matrix kernels on row-major operands (conv_gemm.hip, tgemm.hip): the arguments of a linear layer or an
// implicit-GEMM convolution, and the source of a filter tap.
#pragma once
#include "kernels.h"

namespace df {

struct TileParams {
  // GEMM view
  const bf16_t* A;
  const bf16_t* Wt;
  const float* bias;
  const float* residual;
  const float* chan_add;
  long long chan_ld;
  void* out;
  int M, N, K;
  long long lda, ldw, ldr, ldo;
  int act;
  // convolution geometry (kConv only)
  const bf16_t* top;
  const bf16_t* bot;
  long long halo_bs;
  const bf16_t* left;    // stale column left / right of a vertical strip: pixel (b, row) at left + b*side_bs + row*side_rs
  const bf16_t* right;
  long long side_bs, side_rs;
  int R, W, Cin, Ro, Wo, stride;
  int packed_w;   // W in the tiled layout of launch_pack_weight
  const Scratch* scr;   // host side only: where split-K partials and the page of zeros live
};

// Source pixel (channel 0) of one filter tap: the fresh patch, a stale halo row (patches are horizontal strips) or
// halo column (vertical strips), or nullptr where the tap falls on the zero padding around the image.
template <typename T>
__device__ __forceinline__ const T* conv_tap_src(const T* x, const T* top, const T* bot, long long halo_bs, const T* left,
                                                 const T* right, long long side_bs, long long side_rs, int b, int ri,
                                                 int ci, int R, int W, int Cin) {
  if (ci < 0 || ci >= W) {
    const T* side = ci < 0 ? left : right;
    if (!side || ri < 0 || ri >= R) return nullptr;
    return side + b * side_bs + ri * side_rs;
  }
  if (ri < 0) return top ? top + b * halo_bs + (long long)ci * Cin : nullptr;
  if (ri >= R) return bot ? bot + b * halo_bs + (long long)ci * Cin : nullptr;
  return x + (((long long)b * R + ri) * W + ci) * Cin;
}

// Where an output tile that starts at weight row n0 (a multiple of 32) takes its weights from: elements from the weights to the tile's
// base, bytes from there to the 16 that LDS slot `slot` of tile row `row` receives (rows beyond the last of N: that one, re-read and
// never stored), and bytes from one slab of 64 columns to the next.  LDS row r keeps its 16-byte chunk c at slot c ^ ((r >> 1) & 7).
// Tiled weights hold the rows of a 64 x 64 tile just so, but tile (n / 64, slab) begins at a multiple of 64 rows where a 160-wide output
// tile need not: the base is that of the tile that holds row n0, and the lane counts its rows from there (a tile row 32 further
// has the same swizzle).  The launcher keeps K and ldw below 2^22: the bytes fit 32 bits up to 320 rows row-major, four tiles tiled.
__host__ __device__ inline long long w_tile_base(bool tiled, int n0, int slabs, long long ldw) {
  return tiled ? (long long)(n0 >> 6) * slabs * 4096 : (long long)n0 * ldw;
}
__host__ __device__ inline unsigned int w_lane_bytes(bool tiled, int n0, int row, int slot, int N, int slabs, long long ldw) {
  const unsigned int n = (unsigned int)((n0 + row < N ? n0 + row : N - 1) - (tiled ? n0 & ~63 : n0));
  return 2u * (tiled ? ((n >> 6) * (unsigned int)slabs * 64u + (n & 63u)) * 64u + (unsigned int)slot * 8u
                     : n * (unsigned int)ldw + (unsigned int)(slot ^ ((row >> 1) & 7)) * 8u);
}
__host__ __device__ inline unsigned int w_slab_bytes(bool tiled) { return tiled ? 8192 : 128; }

// Workgroup-tile kernel (tgemm.hip): linear layers and convolutions with K % 64 == 0 (Cin % 64 == 0), N % 4 == 0 and an
// epilogue of whole 16-byte accesses.  DF_ESHAPE if the arguments do not fit.
int launch_tgemm(const TileParams& p, bool conv, int out_dtype, hipStream_t st);
// Convolution of stride 1 with the input pixels kept in LDS over the taps (rconv.hip); the arguments are those launch_tgemm accepts.
int launch_rconv(const TileParams& p, int out_dtype, hipStream_t st);
// Adds the parts of a convolution in their order and finishes it (tgemm.hip).
int launch_conv_reduce(const TileParams& p, const float* partials, int nsplit, int out_dtype, hipStream_t st);

}  // namespace df
