// 16-bit GEMM kernel of the 256 x 256 tile: two groups of four waves that take turns at the matrix cores.
//
// What bounds it: the matrix cores at the clock that power allows, and behind them the operand loads (64 KB per compute unit
// and k-tile).  v_mfma_f32_16x16x32 takes less power per flop than 32x32x16: bare loops of them on N(0, 1) operands run at
// 2036 and 1812 TFLOP/s (2444 and 2453 on constants).
//
// A wave owns 128 x 64 outputs; wave group 0 (waves 0..3, one per SIMD) has the tile's upper 128 rows, group 1 the lower.  A
// k-tile of 64 is two phases of 32 MFMAs: the first 64 of a wave's rows against all its columns, then the other 64 against the
// same column fragments.  A phase is a memory half (fragments out of LDS, loads for later k-tiles) and an MFMA half, with a
// barrier behind each; group 1 runs one barrier behind group 0, so that on every SIMD one wave multiplies while the other
// reads.  What the barriers order:
//   - a part of a stage is loaded again one phase after both groups have read it: A's second rows of k-tile t + 1 in the first
//     phase of t, A's first rows and B of t + 2 in the second phase of t.  Every load has a whole k-tile's time to arrive;
//     the wait behind a memory half lets the NLD youngest of a wave's loads stay in flight.
//   - the waves of group 0 run into the epilogue while group 1 multiplies its last phase.
// With both groups in step, one barrier per k-tile and 32x32x16 the same tile took: 8192^3 876 us (now 722), 32768 x 1024 x 4096
// 222 (193), 32768 x 4096 x 1024 245 (205), both operands K-strided 4096 x 4096 x 8192 266 (192), 1024 x 4096 x 32768 over 4
// splits 293 (219).  Tried: B's loads among the MFMAs (2 % slower), a higher wave priority there (no difference), tiles of
// 256 x 192 (16384 x 768 x 3072, 256 tiles instead of 192: 61 against 63 us) and 256 x 128 (no faster than three stages).
//
// A resident workgroup's loads run on into its next tile: the last two k-tiles of a tile fetch the first ones of the next, the
// epilogue's strips of 16 rows per wave lie behind both stages, and the next tile starts with its operands in LDS.
#pragma once
#include "gemm.h"

template <typename E>
__device__ __forceinline__ f32x4 mfma_16x16x32(bf16x8 a, bf16x8 b, f32x4 c) {
  if constexpr (sizeof(E) == 2 && __is_same(E, fp16)) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(fp16x8, a), __builtin_bit_cast(fp16x8, b), c, 0, 0, 0);
  } else {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
}

template <typename T> struct Vec8 { typedef __attribute__((ext_vector_type(8))) T t; };

// One operand part of a stage: ROWS rows (of A) or columns (of B) x 64 k.  HALF (A): local row r is the tile's row
// (r / 64) * 128 + r % 64, plus what the loads' `extra` bytes come to: the 64 rows of one phase of both wave groups.
//  KC  (memory [rows, K]):  image [row][64]; the 16-byte chunk c of row r sits at slot c ^ ((r >> 1) & 7): the 16 rows of which
//                           a quarter wave reads one chunk lie on 16 different bank groups.
//  !KC (memory [K, rows]):  image [k][rows] as in memory; the 32-byte block b of k-row k sits at slot b ^ (2 (k & 3) + ((k >> 3) & 1)):
//                           the 8 k-rows of which a half wave's transposing read takes one block lie on different banks.
template <int ROWS, bool KC, bool HALF>
struct PPPart {
  static constexpr int BYTES = ROWS * 128;
  static constexpr int PER = ROWS / 64;            // load instructions per wave (8 waves, 1 KiB each)
  static_assert(ROWS == 128 || ROWS == 256, "a k-row of the K-strided image is 256 or 512 bytes");
  uint32_t off;    // this lane's byte offset into the operand at k = 0, first load
  int kc8;         // KC: first k of the lane's chunk
  uint32_t fb[KC ? 2 : 4];  // fragment addresses: KC per k32-step, !KC per 16-row fragment

  __device__ __forceinline__ void init(uint32_t ld, int row0, int wave, int lane) {   // row0: first local row of this wave's fragments
    const int i16 = lane & 15, g = lane >> 4;
    if constexpr (KC) {
      const int r = wave * 8 + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
      kc8 = c * 8;
      off = (uint32_t)r * ld * 2u + (uint32_t)c * 16u;
      fb[0] = (row0 + i16) * 128 + ((g ^ (i16 >> 1)) * 16);
      fb[1] = fb[0] ^ 64;
    } else {
      constexpr int CPR = ROWS / 8, KPI = 64 / CPR;     // chunks per k-row, k-rows per load instruction
      const int k = wave * KPI + lane / CPR, c = (lane % CPR) ^ (((k & 3) << 2) | (((k >> 3) & 1) << 1));
      const int col = HALF ? (c >> 3) * 128 + (c & 7) * 8 : c * 8;
      kc8 = 0;
      off = ((uint32_t)k * ld + (uint32_t)col) * 2u;
      const int R = i16 >> 2, Q = i16 & 3, sw = 2 * R + (g & 1);
      static_for<0, 4>([&](auto f) { fb[f] = (g * 8 + R) * (ROWS * 2) + (((row0 / 16 + decltype(f)::value) ^ sw) * 32) + Q * 8; });
    }
  }
  // the loads of the k-tile that starts at k0; K-contiguous chunks from kend on come as zeros (K-strided rows from kend on
  // are past the descriptor's range)
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rs, uint32_t ld, uint32_t extra, int k0, int kend, char* part, int wave) const {
    uint32_t base = off + (KC ? (uint32_t)k0 * 2u : (uint32_t)k0 * ld * 2u) + extra;
    if (KC && k0 + kc8 >= kend) base = BUF_OOB;
    asm volatile("" : "+v"(base));   // (opaque, or every load of the main loop gets a running offset, and a register, of its own)
    static_for<0, PER>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      const uint32_t step = (uint32_t)(i * (KC ? (HALF ? 128 : 64) : 8 * (64 / (ROWS / 8)))) * ld * 2u;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)(part + (i * 8 + wave) * 1024), 16, (int)(base + step), 0, 0, 0);
    });
  }
  // fragment F (16 rows) of k32-step KK: lane l holds row l % 16, k = 8 (l / 16) .. + 7
  template <int F, int KK>
  __device__ __forceinline__ bf16x8 frag(const char* part) const {
    if constexpr (KC) {
      return *(const bf16x8*)(part + fb[KK] + F * 2048);
    } else {
      typedef __attribute__((ext_vector_type(4))) short s16x4;
      typedef __attribute__((ext_vector_type(8))) short s16x8;
      typedef s16x4 __attribute__((address_space(3))) * lds_ptr;
      const char* p = part + fb[F] + KK * 32 * (ROWS * 2);
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(__attribute__((address_space(3))) char*)p);
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(__attribute__((address_space(3))) char*)(p + 4 * (ROWS * 2)));
      const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      return __builtin_bit_cast(bf16x8, v);
    }
  }
};

__device__ __forceinline__ void buf_store16(u32x4 v, __amdgpu_buffer_rsrc_t r, uint32_t byte_off) {
  __builtin_amdgcn_raw_buffer_store_b128(v, r, (int)byte_off, 0, 0);
}

// A wave's 128 x 64 part of a matrix of T in the epilogue: columns col .. col + n - 1 of row prow + `row`, and with n = 4 the
// same 32 columns on
template <typename T>
struct PPOut {
  __amdgpu_buffer_rsrc_t rs;
  uint32_t lane0, lane1, pitch;   // this lane's byte offsets (out of range where its columns are past N), bytes from row to row
  __device__ __forceinline__ PPOut(T* base, long long ld, int m0, int n0, int M, int N, int prow, int col, int n) {
    const int rows = min(128, M - m0), cols = min(64, N - n0);
    rs = make_rsrc(base + (long long)m0 * ld + n0, rows > 0 && cols > 0 ? (uint32_t)(((rows - 1) * (uint32_t)ld + cols) * sizeof(T)) : 0u);
    pitch = (uint32_t)ld * sizeof(T);
    lane0 = col < cols ? prow * pitch + col * sizeof(T) : BUF_OOB;
    lane1 = n == 4 && col + 32 < cols ? prow * pitch + (col + 32) * sizeof(T) : BUF_OOB;
  }
  __device__ __forceinline__ uint32_t row(int r) const { return (uint32_t)r * pitch; }
  __device__ __forceinline__ uint32_t off(int r) const { return lane0 + row(r); }
};

// epilogue_pass's row through them
template <typename E, typename TC>
struct PPRowIo {
  const GemmArgs& g;
  long long m;
  int ncol, M, N;
  const PPOut<TC>& oc;
  const PPOut<E>& ok;
  int row;
  __device__ __forceinline__ void resid(float (&t)[8]) const {   // (beside a kept activation; no epilogue of the layer has both)
    if (m < M && ncol < N) load8((const E*)g.resid + m * g.ldr + ncol, t);
  }
  __device__ __forceinline__ void old(float (&t)[8]) const {
    
    if constexpr (sizeof(TC) == 4) {
      const f32x4 a = __builtin_bit_cast(f32x4, buf_load16(oc.rs, oc.off(row))), b = __builtin_bit_cast(f32x4, buf_load16(oc.rs, oc.off(row) + 16));
#pragma unroll
      for (int e = 0; e < 4; ++e) { t[e] = a[e]; t[4 + e] = b[e]; }
    } else {
      unpack8<TC>(buf_load16(oc.rs, oc.off(row)), t);
    }
  }
  template <typename T>
  __device__ __forceinline__ static void store(const PPOut<T>& o, int row, const float (&t)[8]) {
    if constexpr (sizeof(T) == 4) {
      buf_store16(__builtin_bit_cast(u32x4, f32x4{t[0], t[1], t[2], t[3]}), o.rs, o.off(row));
      buf_store16(__builtin_bit_cast(u32x4, f32x4{t[4], t[5], t[6], t[7]}), o.rs, o.off(row) + 16);
    } else {
      typename Vec8<T>::t a;
#pragma unroll
      for (int e = 0; e < 8; ++e) a[e] = from_f32<T>(t[e]);
      buf_store16(__builtin_bit_cast(u32x4, a), o.rs, o.off(row));
    }
  }
  __device__ __forceinline__ void keep(const float (&t)[8]) const { store(ok, row, t); }
  __device__ __forceinline__ void put(const float (&t)[8]) const { store(oc, row, t); }
};

constexpr int PP_STAGE = 64 * 1024;                              // A's two parts of 128 rows, B's 256 columns
constexpr int PP_STRIP = 16 * 64 * 4;                            // a wave's epilogue strip: 16 rows of 64 fp32 results
constexpr int PP_LDS = 2 * PP_STAGE + 8 * PP_STRIP;              // the whole LDS of a compute unit

__device__ __forceinline__ void pp_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// EPI as for gemm_mfma_dlds_kernel.
// EPI = EPI_LIVE_SPLITS: fp32 partial results of a K split whose factor follows from the rows that *m_dev says are live
// (live_splits): a grid of LIVE_WGS workgroups, of which tile count x splits have work, one tile each, no epilogue.
constexpr int EPI_LIVE_SPLITS = -2;
// EPI = EPI_SCALED: alpha times the product and nothing else
constexpr int EPI_SCALED = -3;
template <bool AKC, bool BKC, typename TC, typename E, int EPI>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_mfma_pp_kernel(GemmArgs g) {
  constexpr int BM = 256, BN = 256, BK = 64, WM = 128, WN = 64;
  constexpr bool LIVE = EPI == EPI_LIVE_SPLITS;
  const int epi = EPI >= 0 ? EPI : EPI == -1 ? g.epi : 0;
  using PA = PPPart<128, AKC, true>;
  using PB = PPPart<256, BKC, false>;
  static_assert(2 * PA::BYTES + PB::BYTES == PP_STAGE, "stage");
  constexpr int NLD = 2 * PA::PER + PB::PER;       // loads of a wave per k-tile
  extern __shared__ __attribute__((aligned(1024))) char lds[];   // PP_LDS bytes

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;         // (waves w and w + 4 share a SIMD)

  int M = g.M, K = g.K;
  if (g.m_dev) M = min(M, *g.m_dev);
  if (g.k_dev) K = min(K, *g.k_dev);
  const int N = g.N;
  // (the tile order covers the live rows only, so that each XCD gets its share of them: with 4915 of 8192 rows live and
  // the order over all rows, three of the eight XCDs had nothing to do)
  const int tiles_n = (N + BN - 1) / BN, tiles_m = (M + BM - 1) / BM, num_tiles = tiles_m * tiles_n;
  const int nk_all = (K + BK - 1) / BK;
  // A workgroup takes tiles blockIdx.x, blockIdx.x + gridDim.x, ...: launched with one workgroup per tile it runs
  // once, launched with one workgroup per CU it stays resident and walks its share of the tile order.
  int first_tile = blockIdx.x, tile_step = gridDim.x, split = blockIdx.y, per_split = (nk_all + gridDim.y - 1) / gridDim.y;
  long long split_stride = g.split_stride;
  if constexpr (LIVE) {
    const LiveSplits ls = live_splits(M, N, K);
    if ((int)blockIdx.x >= ls.tiles * ls.splits) return;
    first_tile = blockIdx.x % ls.tiles;
    split = blockIdx.x / ls.tiles;
    tile_step = ls.tiles;   // one tile
    per_split = ls.per_split;
    split_stride = ls.stride;
  }
  const int kt0 = split * per_split, kt1 = min(nk_all, kt0 + per_split), nk = kt1 - kt0;
  if (nk <= 0) return;
  const int kend = min(K, kt1 * BK);

  const int z = blockIdx.z, zo = z / g.zdiv, zi = z % g.zdiv;
  const uint32_t lda = (uint32_t)g.lda, ldb = (uint32_t)g.ldb;
  const uint32_t a_half = AKC ? 64u * lda * 2u : 128u;   // from a phase's rows of A to the next phase's
  // buffer descriptors of the operand panels of tile vb (past the last tile: nothing to read)
  const auto panels = [&](int vb, __amdgpu_buffer_rsrc_t& ra, __amdgpu_buffer_rsrc_t& rb) {
    const bool live = vb < num_tiles;
    int tm = 0, tn = 0;
    if (live) tile_of_block(vb, tiles_m, tiles_n, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;
    const bf16* A = (const bf16*)g.A + zo * g.a_zo + zi * g.a_zi + (AKC ? (long long)m0 * g.lda : (long long)m0);
    const bf16* B = (const bf16*)g.B + zo * g.b_zo + zi * g.b_zi + (BKC ? (long long)n0 * g.ldb : (long long)n0);
    ra = make_rsrc(A, live ? tile_bytes<AKC>(g.lda, M - m0, AKC ? K : kend) : 0u);
    rb = make_rsrc(B, live ? tile_bytes<BKC>(g.ldb, N - n0, BKC ? K : kend) : 0u);
  };
  __amdgpu_buffer_rsrc_t ra, rb;   // panels that A's first rows and B are being loaded from
  panels(first_tile, ra, rb);
  bool staged = false;   // the tile's first k-tile, and all of the second but A's second rows, are in the two stages
  int cur_off = 0;       // stage of the k-tile at hand
  for (int vb = first_tile; vb < num_tiles; vb += tile_step) {
  __amdgpu_buffer_rsrc_t ra_next, rb_next, ra1 = ra;   // ra1: the same for A's second rows, which come a phase later
  panels(vb + tile_step, ra_next, rb_next);
  // (computed again for every tile: kept across the epilogues that read a second operand, five or six registers went to
  // scratch, whose reload waits for the tile's stores)
  int lane_ = lane;
  asm volatile("" : "+v"(lane_));
  PA pa;
  PB pb;
  pa.init(lda, wm * 64, wave, lane_);
  pb.init(ldb, wn * WN, wave, lane_);

  f32x4 acc[32];   // [row fragment][column fragment], 16 x 16 each, transposed: lane l holds row l % 16, columns 4 (l / 16) .. + 3
  static_for<0, 32>([&](auto t) { acc[decltype(t)::value] = f32x4{0.f, 0.f, 0.f, 0.f}; });

  if (!staged) {
    char* s0 = lds + cur_off;
    char* s1 = lds + (PP_STAGE - cur_off);
    pa.load(ra, lda, 0u, kt0 * BK, kend, s0, wave);
    pb.load(rb, ldb, 0u, kt0 * BK, kend, s0 + 2 * PA::BYTES, wave);
    pa.load(ra, lda, a_half, kt0 * BK, kend, s0 + PA::BYTES, wave);
    pa.load(ra, lda, 0u, (kt0 + 1) * BK, kend, s1, wave);
    pb.load(rb, ldb, 0u, (kt0 + 1) * BK, kend, s1 + 2 * PA::BYTES, wave);
    wait_vm0();
  }
  pp_barrier();
  if (wm == 1) pp_barrier();
  int kback = 0;   // becomes nk where the loads run on into the next tile
  for (int kt = kt0; kt < kt1; ++kt) {
    char* cur = lds + cur_off;
    char* nxt = lds + (PP_STAGE - cur_off);
    bf16x8 af[8], bfr[8];
    // one MFMA half: row fragments 4 H .. 4 H + 3 against all column fragments
    const auto multiply = [&](auto hc) {
      constexpr int H = decltype(hc)::value;
      static_for<0, 2>([&](auto kk) {
        static_for<0, 16>([&](auto t) {
          constexpr int T = decltype(t)::value, i = T / 4, j = T % 4, q = decltype(kk)::value;
          acc[16 * H + T] = mfma_16x16x32<E>(bfr[q * 4 + j], af[q * 4 + i], acc[16 * H + T]);
        });
      });
    };
    // ---- first phase
    static_for<0, 2>([&](auto kk) {
      constexpr int q = decltype(kk)::value;
      static_for<0, 4>([&](auto i) { af[q * 4 + decltype(i)::value] = pa.template frag<decltype(i)::value, q>(cur); });
      static_for<0, 4>([&](auto j) { bfr[q * 4 + decltype(j)::value] = pb.template frag<decltype(j)::value, q>(cur + 2 * PA::BYTES); });
    });
    if (kt + 1 == kt1) ra1 = ra_next;
    pa.load(ra1, lda, a_half, (kt + 1 == kt1 && nk > 1 ? kt0 : kt + 1) * BK, kend, nxt + PA::BYTES, wave);
    __builtin_amdgcn_sched_barrier(0);
    // (the first k-tile's waits were done ahead of the tile; behind an epilogue they would wait for its stores.  The second
    // k-tile's can be put off as well, with all of it loaded ahead of the stores: no difference)
    if (kt != kt0) asm volatile("s_waitcnt vmcnt(%0)" ::"i"(NLD) : "memory");   // this k-tile's second rows of A are in
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    pp_barrier();
    multiply(std::integral_constant<int, 0>{});
    pp_barrier();
    // ---- second phase
    static_for<0, 2>([&](auto kk) {
      constexpr int q = decltype(kk)::value;
      static_for<0, 4>([&](auto i) { af[q * 4 + decltype(i)::value] = pa.template frag<decltype(i)::value, q>(cur + PA::BYTES); });
    });
    if (kt + 2 == kt1) { ra = ra_next; rb = rb_next; kback = nk; }
    pa.load(ra, lda, 0u, (kt + 2 - kback) * BK, kend, cur, wave);
    pb.load(rb, ldb, 0u, (kt + 2 - kback) * BK, kend, cur + 2 * PA::BYTES, wave);
    __builtin_amdgcn_sched_barrier(0);
    if (kt != kt0) asm volatile("s_waitcnt vmcnt(%0)" ::"i"(NLD) : "memory");   // the next k-tile's first rows of A and its B are in
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    pp_barrier();
    multiply(std::integral_constant<int, 1>{});
    if (wm == 0 || kt + 1 < kt1) pp_barrier();   // (group 1's last one is the one it began with: both count the same)
    cur_off = PP_STAGE - cur_off;
  }
  staged = nk > 1;
  if (!staged) { ra = ra_next; rb = rb_next; }   // a single k-tile: the loads have not run on

  // ---- epilogue -----------------------------------------------------------------------------------
  // 16 rows at a time through the wave's strip: the accumulators' 4 columns x 16 rows per lane go in as one 16-byte store
  // per fragment, rows come out whole.  The 16-byte unit u of row r sits at slot u ^ r: no conflicts either way.
  int tm, tn;
  tile_of_block(vb, tiles_m, tiles_n, tm, tn);
  const int m0 = tm * BM + wm * WM, n0 = tn * BN + wn * WN;
  TC* C = (TC*)g.C + zo * g.c_zo + zi * g.c_zi + (long long)split * split_stride;
  const bool atomic = !LIVE && gridDim.y > 1 && g.split_stride == 0;
  float* strip = (float*)(lds + 2 * PP_STAGE + wave * PP_STRIP);
  const bool vec_ok = gemm_vec_ok(g, epi, C);
  const auto at = [&](int r, int u) { return r * 64 + ((u ^ r) * 4); };
  // a pass is 8 rows, 8 lanes each; a lane keeps its 8 columns through the tile.
  // F4: fp32 results without a 16-bit operand beside them: a lane's columns are two groups of 4, 32 apart, so that each 16-byte
  // store of a wave covers whole 128-byte lines, and its rows are such that the strip's reads do not conflict either
  constexpr bool F4 = sizeof(TC) == 4 && (EPI == 0 || EPI == EPI_BIAS || EPI == EPI_ACCUM || EPI == EPI_SCALED || LIVE);
  const int cc = lane & 7;
  const int prow = F4 ? ((lane >> 3) & 1) * 8 + (lane >> 4) : lane >> 3;   // row of the first pass
  constexpr int PSTEP = F4 ? 4 : 8;                                        // rows from a pass to the next
  const int ncol = n0 + cc * 8;
  // The wave's part of C and of the matrices beside it goes through descriptors that end where its valid rows do, with lanes
  // past N sent out of range: no pass needs a mask.  (Rows so far apart that a part exceeds 2 GiB go through pointers.)
  const bool pre_aux = (epi & (EPI_GELUGRAD | EPI_MULAUX)) != 0, pre_res = !pre_aux && (epi & EPI_RESID);
  constexpr long long FAR = 1LL << 22;
  const bool far = g.ldc >= FAR || ((epi & EPI_GELU) && g.aux_out && g.ldaux >= FAR) || (pre_aux && g.ldaux >= FAR) || ((epi & EPI_RESID) && g.ldr >= FAR);
  const PPOut<TC> oc(C, g.ldc, m0, n0, M, N, prow, cc * (F4 ? 4 : 8), F4 ? 4 : 8);
  const PPOut<E> ok((E*)g.aux_out, g.ldaux, m0, n0, M, N, prow, cc * 8, 8);
  const PPOut<E> op(pre_aux ? (E*)g.aux : (E*)g.resid, pre_aux ? g.ldaux : g.ldr, m0, n0, M, N, prow, cc * 8, 8);
  float bias8[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  float csum8[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (vec_ok && !atomic && !far) {
    if constexpr (F4) {
      if (epi & EPI_BIAS) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int n = n0 + cc * 4 + (e & 3) + (e >> 2) * 32;
          if (n < N) bias8[e] = to_f32(((const E*)g.bias)[n]);
        }
      }
    } else if ((epi & EPI_BIAS) && ncol < N) load8((const E*)g.bias + ncol, bias8);
  }
  const auto strip_order = [] {   // the wave's own LDS traffic executes in order: this is for the compiler
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  const auto park = [&](auto ic) {   // row fragment i into the strip
    constexpr int i = decltype(ic)::value;
    static_for<0, 4>([&](auto jc) {
      constexpr int j = decltype(jc)::value;
      *(f32x4*)(strip + at(lane & 15, j * 4 + (lane >> 4))) = acc[i * 4 + j];
    });
    strip_order();
  };
  if constexpr (EPI == -1 || EPI == EPI_SCALED) {   // (here and not as the strips are filled: two to five registers less)
    if (g.alpha != 1.0f) static_for<0, 32>([&](auto t) { acc[decltype(t)::value] *= g.alpha; });
  }
  park(std::integral_constant<int, 0>{});
  if (vec_ok && !atomic && !far) {
    // The second operand is requested whole, ahead of the first store: loads and stores complete in one order, and a load
    // behind a store would come back after that store has reached the L2, a microsecond or two later while all compute units
    // store.  The 64 registers are the fragments', idle by now.  (32768 x 4096 x 1024 with bias and residual: requested three
    // passes ahead 273 us, now 251; times a kept activation, with column sums 273 and 256.)
    // (Flags read at run time: four passes ahead, or the registers do not suffice for whatever they may say.)
    constexpr int NP = 16, AHEAD = EPI == -1 ? 4 : NP;
    u32x4 pre[AHEAD];
    __builtin_amdgcn_sched_barrier(0);
    if (pre_aux || pre_res) {
      static_for<0, AHEAD>([&](auto qc) { constexpr int q = decltype(qc)::value; pre[q] = buf_load16(op.rs, op.off(q / 2 * 16 + q % 2 * PSTEP)); });
      __builtin_amdgcn_sched_barrier(0);
    }
    // fp32 sums that are added to, two such operands per pass: 8 passes ahead (the head's dE, 30522 x 1024 x 4915: 321 us where
    // each pass asks for its own, now 311)
    if constexpr (F4 && EPI == EPI_ACCUM) {
      static_for<0, NP / 2>([&](auto qc) {
        constexpr int q = decltype(qc)::value, row = q / 2 * 16 + q % 2 * PSTEP;
        pre[2 * q] = buf_load16(oc.rs, oc.lane0 + oc.row(row));
        pre[2 * q + 1] = buf_load16(oc.rs, oc.lane1 + oc.row(row));
      });
      __builtin_amdgcn_sched_barrier(0);
    }
    static_for<0, 8>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      __builtin_amdgcn_sched_barrier(0);
      f32x4 sv[4];
      static_for<0, 2>([&](auto pc) {
        constexpr int p = decltype(pc)::value;
        const int row = prow + p * PSTEP;
        sv[2 * p] = *(const f32x4*)(strip + at(row, F4 ? cc : 2 * cc));
        sv[2 * p + 1] = *(const f32x4*)(strip + at(row, F4 ? cc + 8 : 2 * cc + 1));
      });
      strip_order();
      if constexpr (i + 1 < 8) park(std::integral_constant<int, i + 1>{});   // (under the arithmetic and stores of this one)
      if constexpr (i == 0) {   // the next tile's first stages are in; waited for later they would stand behind the stores
        __builtin_amdgcn_sched_barrier(0);
        if ((F4 && EPI == EPI_ACCUM) || pre_aux || pre_res) asm volatile("s_waitcnt vmcnt(%0)" ::"i"(AHEAD) : "memory");   // (all but the loads just issued)
        else wait_vm0();
        __builtin_amdgcn_sched_barrier(0);
      }
      static_for<0, 2>([&](auto pc) {
        constexpr int p = decltype(pc)::value, row = i * 16 + p * PSTEP;   // row: of the pass, from the wave's first one
        const int m = m0 + row + prow;
        if constexpr (F4) {
          static_for<0, 2>([&](auto hc) {
            constexpr int hf = decltype(hc)::value;
            f32x4 v = sv[2 * p + hf];
            if (epi & EPI_BIAS) v += f32x4{bias8[4 * hf], bias8[4 * hf + 1], bias8[4 * hf + 2], bias8[4 * hf + 3]};
            if constexpr (EPI == EPI_ACCUM) {
              constexpr int q = 2 * i + p, slot = 2 * (q % (NP / 2)) + hf, row2 = (q + NP / 2) / 2 * 16 + (q + NP / 2) % 2 * PSTEP;
              v += __builtin_bit_cast(f32x4, pre[slot]);
              if constexpr (q + NP / 2 < NP) pre[slot] = buf_load16(oc.rs, (hf ? oc.lane1 : oc.lane0) + oc.row(row2));
            }
            buf_store16(__builtin_bit_cast(u32x4, v), oc.rs, (hf ? oc.lane1 : oc.lane0) + oc.row(row));
          });
        } else {
          float v[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] = sv[2 * p + (e >> 2)][e & 3];
          constexpr int q = 2 * i + p, next = q + AHEAD;
          const u32x4 now = pre[q % AHEAD];
          if constexpr (next < NP)
            if (pre_aux || pre_res) pre[q % AHEAD] = buf_load16(op.rs, op.off(next / 2 * 16 + next % 2 * PSTEP));
          epilogue_pass<E>(g, epi, pre_aux, pre_res, now, bias8, v, csum8, m < M, PPRowIo<E, TC>{g, m, ncol, M, N, oc, ok, row});
        }
      });
    });
  } else {
    // splits that add with atomics, rows that are not 16-byte aligned, rows that lie far apart
    wait_vm0();
    static_for<0, 8>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      __builtin_amdgcn_sched_barrier(0);
      const int mrow0 = m0 + i * 16;
      if (atomic) {   // a row of 64 columns per instruction: two cache lines
        if constexpr (sizeof(TC) == 4) {
          float* cp = (float*)C + (long long)mrow0 * g.ldc + n0 + lane;
          const int rows = n0 + lane < N ? min(16, M - mrow0) : 0;
#pragma unroll 1
          for (int row = 0; row < 16; ++row)
            if (row < rows) unsafeAtomicAdd(cp + (long long)row * g.ldc, strip[at(row, lane >> 2) + (lane & 3)]);
        }
      } else if (vec_ok) {
#pragma unroll 1
        for (int p = 0; p < 2; ++p) {
          const int row = (lane >> 3) + p * 8, m = mrow0 + row;
          if (m < M && ncol < N) {
            float v[8], b8[8];
            const f32x4 lo = *(const f32x4*)(strip + at(row, 2 * cc)), hi = *(const f32x4*)(strip + at(row, 2 * cc + 1));
#pragma unroll
            for (int e = 0; e < 4; ++e) { v[e] = lo[e]; v[4 + e] = hi[e]; }
            if (epi & EPI_BIAS) load8((const E*)g.bias + ncol, b8);
            u32x4 pre{};
            if (pre_aux || pre_res) pre = *(const u32x4*)((pre_aux ? (const E*)g.aux + (long long)m * g.ldaux : (const E*)g.resid + (long long)m * g.ldr) + ncol);
            epilogue_pass<E>(g, epi, pre_aux, pre_res, pre, b8, v, csum8, true, RowIo<E, TC>{g, m, ncol, C + (long long)m * g.ldc + ncol});
          }
        }
      } else {
        // (EPI_COLSUM is not served here: the host asks for it only when vec_ok holds)
        const int n = n0 + lane, rows = min(16, M - mrow0);
        if (n < N) {
          const float bias = (epi & EPI_BIAS) ? to_f32(((const E*)g.bias)[n]) : 0.f;
#pragma unroll 1
          for (int row = 0; row < rows; row += 4) {
            float v[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = strip[at(row + r, lane >> 2) + (lane & 3)];
            gemm_epilogue_rows<4, E, TC>(g, epi, C, mrow0 + row, n, min(4, rows - row), bias, v);
          }
        }
      }
      strip_order();
      if constexpr (i + 1 < 8) park(std::integral_constant<int, i + 1>{});
    });
  }
  if ((epi & EPI_COLSUM) && vec_ok && !atomic) {
    // lanes l, l + 8, l + 16, ... hold the same 8 columns (different rows): fold them; the wave's 64 sums go
    // to its own row of the partial-sum matrix (atomics on the few lines of one [N] vector would queue up at L2)
#pragma unroll
    for (int o = 8; o < 64; o <<= 1) {
#pragma unroll
      for (int e = 0; e < 8; ++e) csum8[e] += __shfl_xor(csum8[e], o, WAVE);
    }
    // (a wave whose rows all lie past M has nothing to report, and the partial-sum matrix has no row for it)
    if (lane < 8 && ncol < N && m0 < M) store8(g.colsum + (long long)(m0 / WM) * N + ncol, csum8);
  }
  }
}
