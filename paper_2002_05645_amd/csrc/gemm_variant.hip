// One tile variant of the 16-bit MFMA GEMM (selected with -DL2L_VARIANT=<index>): all four operand
// layouts, 16-bit and fp32 outputs.
#include "gemm.h"
#include "gemm_pp.h"
#include "gemm_variants.h"

#ifndef L2L_VARIANT
#error "compile with -DL2L_VARIANT=<index>"
#endif

namespace {

template <int BM, int BN, int BK, int WM, int WN, bool AKC, bool BKC, typename TC, typename E>
void launch_one(const GemmArgs& g, hipStream_t s, int splits) {
  constexpr int LDS = 2 * (TileLds<BM, BK>::BYTES + TileLds<BN, BK>::BYTES);
  static_assert(LDS <= 160 * 1024, "tile does not fit the 160 KB LDS");
  auto kern = gemm_mfma_kernel<BM, BN, BK, WM, WN, AKC, BKC, TC, E>;
  static const bool once = [&] {
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
    return true;
  }();
  (void)once;
  const int tiles = ((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN);
  dim3 grid(tiles, splits, g.nbatch), block((BM / WM) * (BN / WN) * 64);
  hipLaunchKernelGGL(kern, grid, block, LDS, s, g);
}

template <int BM, int BN, int BK, int WM, int WN, typename TC, typename E>
void launch_layout(const GemmArgs& g, hipStream_t s, int splits) {
  if (g.a_kc && g.b_kc) launch_one<BM, BN, BK, WM, WN, true, true, TC, E>(g, s, splits);
  else if (g.a_kc && !g.b_kc) launch_one<BM, BN, BK, WM, WN, true, false, TC, E>(g, s, splits);
  else if (!g.a_kc && g.b_kc) launch_one<BM, BN, BK, WM, WN, false, true, TC, E>(g, s, splits);
  else launch_one<BM, BN, BK, WM, WN, false, false, TC, E>(g, s, splits);
}

}  // namespace

// NST: LDS stages of gemm_mfma_dlds_kernel, or PP: gemm_mfma_pp_kernel
constexpr int PP = 4;

template <int BM, int BN, int WM, int WN, bool AKC, bool BKC, typename TC, typename E, int NST, int EPI>
constexpr auto direct_kernel() {
  if constexpr (NST == PP) {
    static_assert(BM == 256 && BN == 256 && WM == 128 && WN == 64, "its tile is fixed");
    return gemm_mfma_pp_kernel<AKC, BKC, TC, E, EPI>;
  } else {
    return gemm_mfma_dlds_kernel<BM, BN, WM, WN, AKC, BKC, TC, E, EPI, NST>;
  }
}
template <int BM, int BN, int WM, int WN, int NST>
constexpr int direct_lds_bytes() {
  if constexpr (NST == PP) return PP_LDS;
  else return dlds_lds_bytes<BM, BN, WM, WN, NST>();
}

template <int BM, int BN, int WM, int WN, bool AKC, bool BKC, typename TC, typename E, int NST, int EPI = -1>
void launch_direct_one(const GemmArgs& g, hipStream_t s, int splits) {
  constexpr int LDS = direct_lds_bytes<BM, BN, WM, WN, NST>();
  static_assert(LDS <= 160 * 1024, "tile does not fit the 160 KB LDS");
  auto kern = direct_kernel<BM, BN, WM, WN, AKC, BKC, TC, E, NST, EPI>();
  static const bool once = [&] {
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
    return true;
  }();
  (void)once;
  // (the tiles of which two or four share a compute unit are not made resident: one workgroup per unit would wait for
  // its own loads; 32768 x 4096 x 1024 on 128 x 128 tiles 450 us resident, 322 us with a workgroup per tile)
  const int num_cus = BM == 256 ? g.resident / 8 * 8 : 0;   // a multiple of the 8 XCDs keeps each resident workgroup's tiles on its own XCD's range
  const int tiles = ((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN);
  // more tiles than CUs: one resident workgroup per CU walks the tile order (the kernel's loop)
  const int gx = (num_cus > 0 && splits == 1 && g.nbatch == 1 && tiles > num_cus) ? num_cus : tiles;
  dim3 grid(gx, splits, g.nbatch), block((BM / WM) * (BN / WN) * 64);
  hipLaunchKernelGGL(kern, grid, block, LDS, s, g);
}

// the direct-to-LDS kernels are built for both operands K-contiguous (forward with transposed weights, dX), both K-strided
// (dW) and A K-contiguous with B K-strided
template <int BM, int BN, int WM, int WN, typename TC, typename E, int NST>
void launch_direct(const GemmArgs& g, hipStream_t s, int splits) {
  // 16-bit output and both operands K-contiguous: the layer's forward, recompute and dX GEMMs.  Their eight epilogues
  // get kernels with the flags compiled in (a third off the epilogue's time); any other combination runs the kernel
  // that reads the flags at run time.
  if constexpr (NST == PP) {   // (4096 x 1024 x 1024 with alpha = 0.5: 30.1 us through the flags at run time, now 22.2)
    if (g.a_kc && g.b_kc && g.alpha != 1.0f && g.epi == 0) { launch_direct_one<BM, BN, WM, WN, true, true, TC, E, NST, EPI_SCALED>(g, s, splits); return; }
  }
  if constexpr (sizeof(TC) == 2) {
    if (g.a_kc && g.b_kc && g.alpha == 1.0f) {
      switch (g.epi) {
#define L2L_EPI_CASE(e) case (e): launch_direct_one<BM, BN, WM, WN, true, true, TC, E, NST, (e)>(g, s, splits); return;
        L2L_EPI_CASE(0)
        L2L_EPI_CASE(EPI_BIAS)
        L2L_EPI_CASE(EPI_BIAS | EPI_RESID)
        L2L_EPI_CASE(EPI_BIAS | EPI_GELU)
        L2L_EPI_CASE(EPI_BIAS | EPI_GELU | EPI_KEEPGRAD)
        L2L_EPI_CASE(EPI_MULAUX)
        L2L_EPI_CASE(EPI_MULAUX | EPI_COLSUM)
        L2L_EPI_CASE(EPI_RESID)
#undef L2L_EPI_CASE
        default: break;
      }
    }
  }
  if constexpr (sizeof(TC) == 4 && NST == PP) {
    if (g.live_splits) {   // A K-contiguous, B K-strided: the head's dX
      constexpr int LDS = direct_lds_bytes<BM, BN, WM, WN, NST>();
      auto kern = direct_kernel<BM, BN, WM, WN, true, false, TC, E, NST, EPI_LIVE_SPLITS>();
      static const bool once = [&] {
        (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        return true;
      }();
      (void)once;
      hipLaunchKernelGGL(kern, dim3(LIVE_WGS), dim3((BM / WM) * (BN / WN) * 64), LDS, s, g);
      return;
    }
  }
  // fp32 output: the partial results of K splits and a dW that is stored (no flag), and the logits (bias)
  if constexpr (sizeof(TC) == 4) {
    if (g.alpha == 1.0f && g.a_kc && g.b_kc && g.epi == 0) { launch_direct_one<BM, BN, WM, WN, true, true, TC, E, NST, 0>(g, s, splits); return; }
    if constexpr (BM >= 128)
      if (g.alpha == 1.0f && !g.a_kc && !g.b_kc && g.epi == 0) { launch_direct_one<BM, BN, WM, WN, false, false, TC, E, NST, 0>(g, s, splits); return; }
    if constexpr (NST == PP) {   // a dW or the head's dE added to what is there; the same with K-contiguous operands (7000 x 3072 x 768: 66 us, now 55)
      if (g.alpha == 1.0f && g.a_kc == g.b_kc && g.epi == EPI_ACCUM && !(splits > 1 && g.split_stride == 0)) {
        if (g.a_kc) launch_direct_one<BM, BN, WM, WN, true, true, TC, E, NST, EPI_ACCUM>(g, s, splits);
        else launch_direct_one<BM, BN, WM, WN, false, false, TC, E, NST, EPI_ACCUM>(g, s, splits);
        return;
      }
    }
    if constexpr (NST == PP)
      if (g.alpha == 1.0f && g.a_kc && g.b_kc && g.epi == EPI_BIAS) { launch_direct_one<BM, BN, WM, WN, true, true, TC, E, NST, EPI_BIAS>(g, s, splits); return; }
  }
  if constexpr (BM < 128) {   // built for K-contiguous operands only: callers see to it
    launch_direct_one<BM, BN, WM, WN, true, true, TC, E, NST>(g, s, splits);
  } else {
    if (g.a_kc && g.b_kc) launch_direct_one<BM, BN, WM, WN, true, true, TC, E, NST>(g, s, splits);
    else if (g.a_kc) launch_direct_one<BM, BN, WM, WN, true, false, TC, E, NST>(g, s, splits);
    else launch_direct_one<BM, BN, WM, WN, false, false, TC, E, NST>(g, s, splits);
  }
}

struct TileCfg { int bm, bn, bk, wm, wn, direct; };
#define L2L_ROW(i, bm, bn, bk, wm, wn, d) {bm, bn, bk, wm, wn, d},
constexpr TileCfg kCfg[] = {L2L_GEMM_VARIANTS(L2L_ROW)};
#undef L2L_ROW
constexpr TileCfg kThis = kCfg[L2L_VARIANT];

#define L2L_CAT2(a, b) a##b
#define L2L_CAT(a, b) L2L_CAT2(a, b)
// The element type of the 16-bit operands is fixed per translation unit (-DL2L_ELEM_FP16 selects IEEE half, default
// bfloat16), so that each format's kernels sit in a code object of their own.
#ifdef L2L_ELEM_FP16
typedef fp16 Elem;
#define L2L_LAUNCH_NAME L2L_CAT(l2l_launch_mfma_h, L2L_VARIANT)
#else
typedef bf16 Elem;
#define L2L_LAUNCH_NAME L2L_CAT(l2l_launch_mfma_v, L2L_VARIANT)
#endif

void L2L_LAUNCH_NAME(const GemmArgs& g, hipStream_t s, int splits, bool out_f32) {
  if constexpr (kThis.direct && kThis.bm == 64) {
    if (small_tile_two_stages(g.M, g.N, g.K, g.nbatch, out_f32 ? splits : 1)) {
      if (out_f32) launch_direct<kThis.bm, kThis.bn, kThis.wm, kThis.wn, float, Elem, 2>(g, s, splits);
      else launch_direct<kThis.bm, kThis.bn, kThis.wm, kThis.wn, Elem, Elem, 2>(g, s, 1);
      return;
    }
  }
  if constexpr (kThis.direct) {   // callers pick these variants for every layout pair but (A K-strided, B K-contiguous)
    if (out_f32) launch_direct<kThis.bm, kThis.bn, kThis.wm, kThis.wn, float, Elem, kThis.direct + 1>(g, s, splits);
    else launch_direct<kThis.bm, kThis.bn, kThis.wm, kThis.wn, Elem, Elem, kThis.direct + 1>(g, s, 1);
  } else {
    if (out_f32) launch_layout<kThis.bm, kThis.bn, kThis.bk, kThis.wm, kThis.wn, float, Elem>(g, s, splits);
    else launch_layout<kThis.bm, kThis.bn, kThis.bk, kThis.wm, kThis.wn, Elem, Elem>(g, s, 1);
  }
}
