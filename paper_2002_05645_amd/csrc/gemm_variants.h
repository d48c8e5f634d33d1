// Tile variants of the bf16 MFMA GEMM: X(index, BM, BN, BK, WM, WN, direct).  direct: the kernel
// whose global loads go straight into LDS, 1 with two stages, 2 with three (the 64 x 64 tile: both operands K-contiguous only, with three or two),
// 3 the kernel whose two wave groups take turns at the matrix cores.  Each variant is compiled
// in its own translation unit (gemm_variant.hip with -DL2L_VARIANT=index) so that the build runs in parallel.
#pragma once
#include <hip/hip_runtime.h>
#include "common.h"

#define L2L_GEMM_VARIANTS(X) \
  X(0, 128, 128, 64, 64, 64, 0) \
  X(1, 128, 64, 64, 64, 32, 0) \
  X(2, 256, 128, 64, 64, 64, 0) \
  X(3, 256, 256, 64, 128, 64, 0) \
  X(4, 128, 128, 64, 64, 64, 2) \
  X(5, 64, 64, 64, 32, 32, 2) \
  X(6, 256, 256, 64, 128, 64, 3) \
  X(7, 128, 128, 64, 64, 64, 1) \
  X(8, 256, 128, 64, 64, 64, 2)

constexpr int kNumGemmVariants = 9;

// 64 x 64 tiles: whether two LDS stages are faster than three, which hide the way to memory but of which three workgroups and
// not four share a compute unit.  They are with less than six k-tiles where units have more than one workgroup (bias and residual,
// two and three stages: 7000 x 512 x 128 7.5 and 8.8 us, 4096 x 1024 x 256 9.0 and 10.2, 16384 x 1280 x 320 35.9 and 37.8; but
// 8192 x 768 x 768 21.6 and 19.6, 5000 x 1024 x 1024 24.2 and 20.5, and a layer of 256 columns forward, 64 tokens, 33.0 and 32.1),
// and where the launch fits the chip with four workgroups per unit but not with three (4096 x 1024 x 1024 16.6 and 18.1,
// 7000 x 512 x 512 10.4 and 11.7; with 32 k-tiles no difference).
inline bool small_tile_two_stages(int M, int N, int K, int nbatch, int splits) {
  const int k_tiles = ((K + 63) / 64 + splits - 1) / splits;
  const long long blocks = (long long)((M + 63) / 64) * ((N + 63) / 64) * splits * nbatch;
  return blocks > 256 && (k_tiles < 6 || (k_tiles < 24 && blocks > 3 * 256 && blocks <= 4 * 256));
}

// launches variant `index` (layouts and output type taken from the arguments)
#define L2L_DECLARE(i, bm, bn, bk, wm, wn, d)                                                      \
  void l2l_launch_mfma_v##i(const GemmArgs& g, hipStream_t s, int splits, bool out_f32); /* bf16 */ \
  void l2l_launch_mfma_h##i(const GemmArgs& g, hipStream_t s, int splits, bool out_f32); /* fp16 */
L2L_GEMM_VARIANTS(L2L_DECLARE)
#undef L2L_DECLARE
