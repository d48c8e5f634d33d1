// fp32 GEMM on the matrix cores (v_mfma_f32_32x32x2_f32: fp32 operands, fp32 accumulate).
#pragma once
#include "gemm.h"

// Block tile 64 x 64, k-tiles of 32, four waves of 32 x 32.  Bound by the matrix cores: a k-tile's 16 products take a SIMD
// 1024 clocks and its operands are 16 KB, half of what a compute unit can load meanwhile.  So nothing elaborate feeds
// them: a k-tile goes global -> registers -> LDS, requested two k-tiles ahead (a k-tile's products take half of what a load
// from memory does; one ahead the layer of width 768 took 2443 us, two ahead 2281, a step of the tiny model 1265 and 1140), in two
// stages of 18 KB, and the other workgroups of the unit (four fit) cover the waits.  (A 128 x 128 tile, two workgroups per unit, took 257 us where this one takes 185
// at 19.3 GFLOP: three of its workgroups per unit leave the last one alone with its own waits.)
// The order of the contraction index is free as long as both operands agree: lane half h supplies k = 8 s + 4 h + j in
// product j of step s, which lets a K-contiguous operand be read from its [row][32] image as one 16-byte fragment per
// step (pitch 36: 16 rows on 16 different bank groups) and a K-strided one from its [k][rows] image as four dwords
// (pitch rows + 8: the two lane halves on different banks).  No operand is transposed, whatever its layout in memory.
// Results leave straight from the accumulators: a register holds 32 consecutive columns of two rows, which are whole
// 128-byte segments in fp32.
// Measured (4096 tokens of width 768): 105 to 118 TFLOP/s against 22 to 45 with the vector-ALU kernel it replaces (dW of
// 768 x 3072: 878 -> 185 us; out-projection 446 -> 51 us), of 154 that a library product of 8192^3 reaches.
constexpr int F32_TILE = 64;

template <int ROWS, bool KC>
struct F32Tile {
  static constexpr int BK = 32;
  static constexpr int PITCH = KC ? BK + 4 : ROWS + 8;            // floats
  static constexpr int FLOATS = KC ? ROWS * PITCH : BK * PITCH;   // one stage
  static constexpr int PER = ROWS * BK / 4 / 256;                 // 16-byte chunks per thread
  u32x4 r[PER];

  // byte range of the panel seen from its first element, whole 16-byte chunks
  static __device__ __forceinline__ uint32_t bytes(long long ld, int rows_left, int K) {
    const long long k4 = (K + 3) & ~3, r4 = (rows_left + 3) & ~3;
    return (uint32_t)((KC ? (long long)(rows_left - 1) * ld + k4 : (long long)(K - 1) * ld + r4) * 4);
  }
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rs, uint32_t ld, int k0, int K, int tid) {
    static_for<0, PER>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      const int u = tid + i * 256;
      if constexpr (KC) {
        const int row = u / 8, k = k0 + (u % 8) * 4;
        const uint32_t off = ((uint32_t)row * ld + (uint32_t)k) * 4u;
        r[i] = buf_load16(rs, k < K ? off : BUF_OOB);
        if (K & 3) {   // a chunk that straddles K: what lies behind it in memory is not part of the operand
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (k + e >= K) r[i][e] = 0u;
        }
      } else {   // rows k >= K lie past the descriptor's range and read as zero
        const int k = u / (ROWS / 4), c = u % (ROWS / 4);
        r[i] = buf_load16(rs, ((uint32_t)(k0 + k) * ld + (uint32_t)(c * 4)) * 4u);
      }
    });
  }
  __device__ __forceinline__ void store(float* lds, int tid) const {
    static_for<0, PER>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      const int u = tid + i * 256;
      if constexpr (KC) *(u32x4*)(lds + (u / 8) * PITCH + (u % 8) * 4) = r[i];
      else *(u32x4*)(lds + (u / (ROWS / 4)) * PITCH + (u % (ROWS / 4)) * 4) = r[i];
    });
  }
  // the four k of step s that this lane's half supplies, for row / column `row`
  static __device__ __forceinline__ f32x4 frag(const float* lds, int row, int s, int lane) {
    const int k = s * 8 + (lane >> 5) * 4;
    if constexpr (KC) {
      return *(const f32x4*)(lds + row * PITCH + k);
    } else {
      const float* p = lds + k * PITCH + row;
      return f32x4{p[0], p[PITCH], p[2 * PITCH], p[3 * PITCH]};
    }
  }
};

// grid: (tiles, K splits, batch).  With splits, split s stores its partial result at C + s * split_stride (also where it
// has no k-tile of its own: zeros), and the caller adds them up.
template <bool AKC, bool BKC>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmArgs g) {
  constexpr int BM = F32_TILE, BN = F32_TILE, BK = 32;
  using TA = F32Tile<BM, AKC>;
  using TB = F32Tile<BN, BKC>;
  constexpr int STAGE = TA::FLOATS + TB::FLOATS;
  extern __shared__ __attribute__((aligned(16))) float ldsf[];   // 2 * STAGE floats

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / 2, wn = wave % 2;
  int M = g.M, K = g.K;
  if (g.m_dev) M = min(M, *g.m_dev);
  if (g.k_dev) K = min(K, *g.k_dev);
  const int N = g.N;
  const int tiles_n = (N + BN - 1) / BN, tiles_m = (M + BM - 1) / BM;
  if ((int)blockIdx.x >= tiles_m * tiles_n) return;   // (the tile order covers the live rows, dealt out over the XCDs)
  int tm, tn;
  tile_of_block(blockIdx.x, tiles_m, tiles_n, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const int nk_all = (K + BK - 1) / BK;
  const int per_split = (nk_all + gridDim.y - 1) / gridDim.y;
  const int kt0 = blockIdx.y * per_split, kt1 = min(nk_all, kt0 + per_split);

  const int z = blockIdx.z, zo = z / g.zdiv, zi = z % g.zdiv;
  const float* A = (const float*)g.A + zo * g.a_zo + zi * g.a_zi + (AKC ? (long long)m0 * g.lda : (long long)m0);
  const float* B = (const float*)g.B + zo * g.b_zo + zi * g.b_zi + (BKC ? (long long)n0 * g.ldb : (long long)n0);
  float* C = (float*)g.C + zo * g.c_zo + zi * g.c_zi + (long long)blockIdx.y * g.split_stride;

  f32x16 acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (kt0 < kt1) {
    const __amdgpu_buffer_rsrc_t ra = make_rsrc(A, TA::bytes(g.lda, M - m0, K));
    const __amdgpu_buffer_rsrc_t rb = make_rsrc(B, TB::bytes(g.ldb, N - n0, K));
    const uint32_t lda = (uint32_t)g.lda, ldb = (uint32_t)g.ldb;
    TA ta[2];
    TB tb[2];
    const auto load = [&](auto pc, int kt) {
      constexpr int P = decltype(pc)::value;
      ta[P].load(ra, lda, kt * BK, K, tid);
      tb[P].load(rb, ldb, kt * BK, K, tid);
    };
    const auto store = [&](auto pc) {   // register set P goes to stage P
      constexpr int P = decltype(pc)::value;
      ta[P].store(ldsf + P * STAGE, tid);
      tb[P].store(ldsf + P * STAGE + TA::FLOATS, tid);
    };
    constexpr std::integral_constant<int, 0> even{};
    constexpr std::integral_constant<int, 1> odd{};
    load(even, kt0);
    if (kt0 + 1 < kt1) load(odd, kt0 + 1);
    store(even);
    __syncthreads();
    const int arow = wm * 32 + (lane & 31), brow = wn * 32 + (lane & 31);
    const auto step = [&](auto pc, int kt) {
      constexpr int P = decltype(pc)::value;
      const float* cur = ldsf + P * STAGE;
      if (kt + 2 < kt1) load(pc, kt + 2);   // (set P held k-tile kt, which is in LDS)
      static_for<0, BK / 8>([&](auto sc) {
        constexpr int s = decltype(sc)::value;
        const f32x4 af = TA::frag(cur, arow, s, lane), bf = TB::frag(cur + TA::FLOATS, brow, s, lane);
        static_for<0, 4>([&](auto ec) {
          constexpr int e = decltype(ec)::value;
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(af[e], bf[e], acc, 0, 0, 0);
        });
      });
      if (kt + 1 < kt1) store(std::integral_constant<int, P ^ 1>{});   // (the other stage was last read before the previous barrier)
      __syncthreads();
    };
    for (int kt = kt0; kt < kt1; kt += 2) {
      step(even, kt);
      if (kt + 1 < kt1) step(odd, kt + 1);
    }
  }
  // Register r of a lane: row 8 (r / 4) + 4 (lane / 32) + r % 4, column lane % 32.  What the epilogue reads is asked for
  // 16 rows at a time, ahead of the first store: element by element (gemm_epilogue) every load would wait behind the
  // previous element's store, which may alias it for all the compiler knows.
  const int epi = g.epi;
  const int n = n0 + wn * 32 + (lane & 31), mb = m0 + wm * 32 + 4 * (lane >> 5);
  if (n >= N) return;
  const auto row = [&](int r) { return (long long)(mb + 8 * (r >> 2) + (r & 3)); };
  const auto fetch = [&](const void* p, long long ld, float (&d)[16]) {
#pragma unroll
    for (int r = 0; r < 16; ++r) d[r] = row(r) < M ? ((const float*)p)[row(r) * ld + n] : 0.f;
  };
  float aux[16], res[16], old[16];
  const float bias = (epi & EPI_BIAS) ? ((const float*)g.bias)[n] : 0.f;
  if (epi & (EPI_GELUGRAD | EPI_MULAUX)) fetch(g.aux, g.ldaux, aux);
  if (epi & EPI_RESID) fetch(g.resid, g.ldr, res);
  if (epi & EPI_ACCUM) fetch(C, g.ldc, old);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    if (row(r) >= M) continue;
    float v = g.alpha * acc[r] + bias;
    if (epi & EPI_GELU) {
      if (g.aux_out) ((float*)g.aux_out)[row(r) * g.ldaux + n] = (epi & EPI_KEEPGRAD) ? gelu_grad_f(v) : v;
      v = gelu_f(v);
    }
    if (epi & EPI_GELUGRAD) v *= gelu_grad_f(aux[r]);
    if (epi & EPI_MULAUX) v *= aux[r];
    if (epi & EPI_RESID) v += res[r];
    if (epi & EPI_ACCUM) v += old[r];
    C[row(r) * g.ldc + n] = v;
  }
}
