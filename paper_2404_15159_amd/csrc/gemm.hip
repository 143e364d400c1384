// GEMM engine of libmixlora:  C[M,N] = sum_s A_s[M,K_s] * B_s[N,K_s]^T  ("NT", K contiguous).
//
// bf16 storage: the frozen projections of more than 128 rows run on gemm_bf16_pp_kernel (256-wide
// tiles, two groups of four waves taking turns at the matrix pipe and at memory, trailing tiles
// cut along K); few rows (decode) on gemm_bf16_few_kernel's narrow tiles, or cut along K on the large
// ones where a contraction is ragged or the columns are few; one and two rows, and up to four into few
// columns, on the matrix-vector kernel gemm_bf16_rows_kernel; what none of them takes on the
// register-staged gemm_bf16_kernel.  XCD-aware + grouped tile order everywhere, so that the tiles
// resident on one XCD share operand rows in that XCD's L2.
// fp32 storage: MFMA 16x16x4 tiles with K spread over the waves (gemm_f32_kernel; the fp32
// configuration is a small parity case).
//
// Every frozen projection of the block (shared gate/up: Algorithm 1 lines 7-8; down: line 14)
// and their transposes in the backward go through here; LoRA terms enter either as extra
// K segments (low-rank K-extension) or through the element-wise kernels.
#include "common.h"

#include <type_traits>

namespace mixlora {

struct GemmBatch {
  GemmProblem p[GEMM_MAX_PROBLEMS];
};

// Logical id of block `bid` of a run of `nb` consecutive blocks: blocks that land on the same XCD
// (the hardware deals them out in turn, so equal bid % 8) get consecutive logical ids.
__device__ __forceinline__ int xcd_order(int bid, int nb) {
  const int q = nb >> 3, rem = nb & 7;
  const int xcd = bid & 7, local = bid >> 3;
  return xcd * q + (xcd < rem ? xcd : rem) + local;
}
// Tile of a logical id: consecutive ids walk GROUP tile-rows at a time.
__device__ __forceinline__ void tile_of_lid(int lid, int tiles_m, int tiles_n, int &tm, int &tn) {
  constexpr int GROUP = 4;   // measured: 4 slightly ahead of 2, 8, 16 (all within 3 %)
  const int width = GROUP * tiles_n;
  const int group_id = lid / width;
  const int first_m = group_id * GROUP;
  const int gsz = (tiles_m - first_m) < GROUP ? (tiles_m - first_m) : GROUP;
  const int in_group = lid - group_id * width;
  tm = first_m + in_group % gsz;
  tn = in_group / gsz;
}

// Both steps for a grid that holds the tiles of one problem only.
__device__ __forceinline__ void tile_of_block(int bid, int tiles_m, int tiles_n, int &tm, int &tn) {
  tile_of_lid(xcd_order(bid, tiles_m * tiles_n), tiles_m, tiles_n, tm, tn);
}

template <typename OutT> __device__ __forceinline__ void store_c(OutT *p, float v);
template <> __device__ __forceinline__ void store_c<float>(float *p, float v) { *p = v; }
template <> __device__ __forceinline__ void store_c<bf16_t>(bf16_t *p, float v) { *p = (bf16_t)v; }

template <typename OutT>
__device__ __forceinline__ void store_c4(OutT *p, float a, float b, float c, float d);
template <> __device__ __forceinline__ void store_c4<float>(float *p, float a, float b, float c, float d) {
  *reinterpret_cast<float4 *>(p) = make_float4(a, b, c, d);
}
template <> __device__ __forceinline__ void store_c4<bf16_t>(bf16_t *p, float a, float b, float c, float d) {
  typedef bf16_t bf16x4v_t __attribute__((ext_vector_type(4)));
  bf16x4v_t v;
  v[0] = (bf16_t)a; v[1] = (bf16_t)b; v[2] = (bf16_t)c; v[3] = (bf16_t)d;
  *reinterpret_cast<bf16x4v_t *>(p) = v;
}

template <int BM, int BN, int BK, int WGM, int WGN, typename OutT>
__global__ __launch_bounds__(WGM *WGN * 64) void gemm_bf16_kernel(GemmBatch args) {
  constexpr int NT = WGM * WGN * 64;
  constexpr int LD = BK + 8;        // LDS row pitch in elements: 16 bytes of padding per row
  constexpr int CPR = BK / 8;       // 16-byte chunks per tile row
  constexpr int RPP = NT / CPR;     // tile rows covered by one pass of all threads
  constexpr int A_IT = BM / RPP, B_IT = BN / RPP;
  constexpr int TM = BM / WGM, TN = BN / WGN, MI = TM / 32, NI = TN / 32;
  static_assert(BM % RPP == 0 && BN % RPP == 0, "tile/threads mismatch");
  static_assert(TM % 32 == 0 && TN % 32 == 0 && BK % 16 == 0, "wave tile");

  extern __shared__ __align__(16) unsigned char smem[];
  bf16_t *As = reinterpret_cast<bf16_t *>(smem);   // [2][BM][LD]
  bf16_t *Bs = As + 2 * BM * LD;                   // [2][BN][LD]

  const GemmProblem &P = args.p[blockIdx.z];
  const int M = P.M, N = P.N;
  const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
  int tm, tn;
  tile_of_block(blockIdx.x, tiles_m, tiles_n, tm, tn);
  const int row0 = tm * BM, col0 = tn * BN;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;
  const int kc = tid % CPR;         // this thread's 16-byte chunk within a tile row
  const int r_in = tid / CPR;       // first tile row this thread loads

  f32x16_t acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; i++)
#pragma unroll
    for (int j = 0; j < NI; j++)
#pragma unroll
      for (int e = 0; e < 16; e++) acc[i][j][e] = 0.f;

  // Global -> register prefetch.  Rows/columns past the matrix edge are clamped to the last
  // valid one: their products land in C rows/columns that are never stored.  K chunks past
  // the segment's end are loaded from a valid address and replaced by zeros.
  uint4 ra[A_IT], rb[B_IT];
  const bf16_t *pa[A_IT], *pb[B_IT];
  int Kcur = 0;
  auto setup = [&](int s) {
    const GemmSeg &S = P.seg[s];
    const bf16_t *Ab = reinterpret_cast<const bf16_t *>(S.A) + kc * 8;
    const bf16_t *Bb = reinterpret_cast<const bf16_t *>(S.B) + kc * 8;
#pragma unroll
    for (int i = 0; i < A_IT; i++) {
      int r = row0 + r_in + i * RPP;
      r = r < M ? r : M - 1;
      pa[i] = Ab + (int64_t)r * S.lda;
    }
#pragma unroll
    for (int i = 0; i < B_IT; i++) {
      int c = col0 + r_in + i * RPP;
      c = c < N ? c : N - 1;
      pb[i] = Bb + (int64_t)c * S.ldb;
    }
    Kcur = S.K;
  };
  auto gload = [&](int k0) {
    const bool kok = k0 + kc * 8 < Kcur;
    const int ko = kok ? k0 : 0;
#pragma unroll
    for (int i = 0; i < A_IT; i++) {
      const uint4 v = *reinterpret_cast<const uint4 *>(pa[i] + ko);
      ra[i] = kok ? v : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < B_IT; i++) {
      const uint4 v = *reinterpret_cast<const uint4 *>(pb[i] + ko);
      rb[i] = kok ? v : make_uint4(0, 0, 0, 0);
    }
  };
  auto lstore = [&](int buf) {
    bf16_t *a = As + buf * BM * LD, *b = Bs + buf * BN * LD;
#pragma unroll
    for (int i = 0; i < A_IT; i++)
      *reinterpret_cast<uint4 *>(a + (r_in + i * RPP) * LD + kc * 8) = ra[i];
#pragma unroll
    for (int i = 0; i < B_IT; i++)
      *reinterpret_cast<uint4 *>(b + (r_in + i * RPP) * LD + kc * 8) = rb[i];
  };

  const int nseg_total = P.nseg;
  int total_tiles = 0;
  for (int s = 0; s < nseg_total; s++) total_tiles += (P.seg[s].K + BK - 1) / BK;

  int seg = 0, k0 = 0;   // position of the tile being prefetched
  setup(0);
  gload(0);
  lstore(0);
  __syncthreads();
  int buf = 0;
  const bf16_t *a_rd = As + (wm * TM + (lane & 31)) * LD + (lane >> 5) * 8;
  const bf16_t *b_rd = Bs + (wn * TN + (lane & 31)) * LD + (lane >> 5) * 8;
  for (int it = 0; it < total_tiles; it++) {
    const bool more = it + 1 < total_tiles;
    if (more) {
      k0 += BK;
      if (k0 >= Kcur) {   // next segment (rare)
        seg++;
        setup(seg);
        k0 = 0;
      }
      gload(k0);
    }
    const bf16_t *a = a_rd + buf * BM * LD;
    const bf16_t *b = b_rd + buf * BN * LD;
#pragma unroll
    for (int kk = 0; kk < BK; kk += 16) {
      bf16x8_t af[MI], bfr[NI];
#pragma unroll
      for (int i = 0; i < MI; i++) af[i] = *reinterpret_cast<const bf16x8_t *>(a + i * 32 * LD + kk);
#pragma unroll
      for (int j = 0; j < NI; j++) bfr[j] = *reinterpret_cast<const bf16x8_t *>(b + j * 32 * LD + kk);
#pragma unroll
      for (int i = 0; i < MI; i++)
#pragma unroll
        for (int j = 0; j < NI; j++)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
    }
    if (more) {
      lstore(buf ^ 1);
      __syncthreads();
      buf ^= 1;
    }
  }

  // C fragment of a 32x32 block: column = lane % 32, row = 8*(e/4) + 4*(lane/32) + e%4
  OutT *C = reinterpret_cast<OutT *>(P.C);
  const int cbase = col0 + wn * TN + (lane & 31);
  const int rbase = row0 + wm * TM + (lane >> 5) * 4;
#pragma unroll
  for (int i = 0; i < MI; i++)
#pragma unroll
    for (int j = 0; j < NI; j++) {
      const int c = cbase + j * 32;
      if (c < N) {
#pragma unroll
        for (int e = 0; e < 16; e++) {
          const int r = rbase + i * 32 + (e >> 2) * 8 + (e & 3);
          if (r < M) store_c<OutT>(C + (int64_t)r * P.ldc + c, acc[i][j][e]);
        }
      }
    }
}

// ---- bf16, direct to LDS ------------------------------------------------------------------------
// Operand tiles go from global memory straight into LDS (global_load_lds_dwordx4: lane i's 16 bytes
// land at M0 + 16*i, no VGPR round trip) through a ring, so that several K tiles are in flight while
// one is consumed.  LDS rows are unpadded (the DMA writes 1 KiB contiguous per wave instruction); bank
// conflicts of the 128-bit fragment reads are avoided by an XOR swizzle of the 16-byte chunk index with
// the row's 256-byte bank-row number, applied on the global-address side of the copy.
// The loads and their s_waitcnt are inline asm: the compiler's own bookkeeping would wait for
// all outstanding LDS DMA before every LDS read and collapse the ring to depth one.
// Requires operands below 4 GiB (32-bit lane offsets).
__device__ __forceinline__ void dma16(uint32_t voff, const void *sbase, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(voff), "s"(sbase), "s"(lds_addr)
               : "memory", "m0");
}
// the same, streaming: for data that this launch reads once
__device__ __forceinline__ void dma16_nt(uint32_t voff, const void *sbase, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt"
               :
               : "v"(voff), "s"(sbase), "s"(lds_addr)
               : "memory", "m0");
}
template <int N> __device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}
__device__ __forceinline__ const void *uniform_ptr(const void *p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<const void *>(((uint64_t)hi << 32) | lo);
}

// ---- bf16, few rows: one row tile, narrow column tiles -------------------------------------------
// Up to 128 rows (decode): bound by streaming the weights once.  One tile holds all rows (BM = 32, 64 or
// 128) and BN weight rows, four waves two by two, MFMA 16x16x32, a ring of four 64-wide K tiles.  What
// sets the rate is how many times the activations go through the L2s beside the weights (once per
// column tile: with 64-column tiles as much as the weights themselves) and how many CUs stream: the
// tiles are as wide as still leaves one for nearly every CU (few_width below).  64 tokens of the
// 7B block, gate and up projections: 349 tiles of 64 columns 44.6 us, 177 of 128 37.4, 233 of 96 36.0
// (5.0 TB/s); a token's own matrix-vector kernel, which has no second operand to fetch, 31.7.  Without
// effect there: rings of 4 to 9 tiles, K tiles of 128.
// Requires whole K tiles.
template <int MAX, int PER> __device__ __forceinline__ void wait_tiles(int n) {   // all but min(n, MAX) groups
  if constexpr (MAX == 0) {
    wait_vmcnt<0>();
  } else {
    if (n >= MAX) wait_vmcnt<MAX * PER>();
    else wait_tiles<MAX - 1, PER>(n);
  }
}
struct FewPlan {
  int nprob, tiles, streaming;       // streaming: the weights (B, read once by this launch) bypass the caches
  int start[GEMM_MAX_PROBLEMS];      // first block of every problem
};

template <int BM, int BN, int STAGES>
__global__ __launch_bounds__(256) void gemm_bf16_few_kernel(GemmBatch args, FewPlan plan, FewRank rk) {
  constexpr int BK = 64, ROWB = BK * 2;
  constexpr int IA = BM / 32, IB = BN / 32, IPW = IA + IB;   // 1 KiB pieces (8 rows) per wave and K tile
  constexpr int STAGE = (BM + BN) * ROWB;
  constexpr int TM = BM / 2, TN = BN / 2, MI = TM / 16, NI = TN / 16;
  static_assert(BM % 32 == 0 && BN % 32 == 0 && STAGES >= 2 && (STAGES - 2) * IPW < 64, "tile shape");

  extern __shared__ __align__(16) unsigned char smem[];
  const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char *)smem;
  if ((int)blockIdx.x >= plan.tiles) {   // behind the tiles: the rank term's sums, a token each
    float *sq = reinterpret_cast<float *>(smem), *red = sq + FEW_RANK_SUMS;
    const int t = blockIdx.x - plan.tiles;
    few_rank_sums(rk, t, true, 256, red, sq);
    if ((int)threadIdx.x < rk.k * rk.r) rk.sums[t * FEW_RANK_SUMS + threadIdx.x] = sq[threadIdx.x];
    return;
  }
  int pi = 0;
  while (pi + 1 < plan.nprob && plan.start[pi + 1] <= (int)blockIdx.x) pi++;
  const GemmProblem &P = args.p[pi];
  const int M = P.M, N = P.N, col0 = ((int)blockIdx.x - plan.start[pi]) * BN;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;

  f32x4_t acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; i++)
#pragma unroll
    for (int j = 0; j < NI; j++) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const int lrow = lane >> 3, lpos = lane & 7;
  uint32_t offA[IA], offB[IB];
  const unsigned char *baseA = nullptr, *baseB = nullptr;
  int seg = 0, k0 = 0, Kcur = 0, issued = 0, total = 0;
  for (int sgi = 0; sgi < P.nseg; sgi++) total += P.seg[sgi].K / BK;
  auto setup = [&]() {
    const GemmSeg &S = P.seg[seg];
#pragma unroll
    for (int j = 0; j < IA; j++) {
      const int q = (wave + 4 * j) * 8 + lrow, rr = q < M ? q : M - 1;
      offA[j] = (uint32_t)rr * (uint32_t)S.lda * 2u + (lpos ^ ((q >> 1) & 7)) * 16;
    }
#pragma unroll
    for (int j = 0; j < IB; j++) {
      const int q = (wave + 4 * j) * 8 + lrow, c = col0 + q < N ? col0 + q : N - 1;
      offB[j] = (uint32_t)c * (uint32_t)S.ldb * 2u + (lpos ^ ((q >> 1) & 7)) * 16;
    }
    baseA = reinterpret_cast<const unsigned char *>(S.A);
    baseB = reinterpret_cast<const unsigned char *>(S.B);
    Kcur = S.K;
  };
  setup();
  auto issue_next = [&]() {   // copies of tile number `issued` (if there is one) into its ring slot
    if (issued < total) {
      if (k0 >= Kcur) {
        seg++;
        setup();
        k0 = 0;
      }
      const void *ga = uniform_ptr(baseA + (size_t)k0 * 2), *gb = uniform_ptr(baseB + (size_t)k0 * 2);
      const uint32_t la = lds0 + (issued % STAGES) * STAGE + wave * 1024, lb = la + BM * ROWB;
#pragma unroll
      for (int j = 0; j < IA; j++) dma16(offA[j], ga, la + j * 4096);
      if (plan.streaming) {
#pragma unroll
        for (int j = 0; j < IB; j++) dma16_nt(offB[j], gb, lb + j * 4096);
      } else {
#pragma unroll
        for (int j = 0; j < IB; j++) dma16(offB[j], gb, lb + j * 4096);
      }
      k0 += BK;
    }
    issued++;
  };
#pragma unroll
  for (int s0 = 0; s0 < STAGES - 1; s0++) issue_next();

  const int l15 = lane & 15, hi = lane >> 4;
  const int koff[2] = {(hi ^ (l15 >> 1)) * 16, ((4 + hi) ^ (l15 >> 1)) * 16};   // swizzled chunks
  const unsigned char *a_rd = smem + (wm * TM + l15) * ROWB;
  const unsigned char *b_rd = smem + BM * ROWB + (wn * TN + l15) * ROWB;
  for (int it = 0; it < total; it++) {
    wait_tiles<STAGES - 2, IPW>(total - 1 - it);   // tile `it` has landed, up to STAGES - 2 newer ones fly on
    __syncthreads();
    issue_next();   // refills the slot that tile it-1 occupied: every wave is past reading it
    const int st = (it % STAGES) * STAGE;
#pragma unroll
    for (int ks = 0; ks < 2; ks++) {
      bf16x8_t fa[MI], fb[NI];
#pragma unroll
      for (int i = 0; i < MI; i++)
        fa[i] = *reinterpret_cast<const bf16x8_t *>(a_rd + st + i * 16 * ROWB + koff[ks]);
#pragma unroll
      for (int j = 0; j < NI; j++)
        fb[j] = *reinterpret_cast<const bf16x8_t *>(b_rd + st + j * 16 * ROWB + koff[ks]);
#pragma unroll
      for (int i = 0; i < MI; i++)
#pragma unroll
        for (int j = 0; j < NI; j++)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
    }
  }
  // a lane holds 4 consecutive columns of a row
  auto store = [&](auto *C) {
    typedef typename std::remove_pointer<decltype(C)>::type OutT;
    const bool whole = (P.ldc & 3) == 0 && (reinterpret_cast<uintptr_t>(C) & 15) == 0;
#pragma unroll
    for (int i = 0; i < MI; i++) {
      const int r = wm * TM + i * 16 + l15;
      if (r >= M) continue;
#pragma unroll
      for (int j = 0; j < NI; j++) {
        const int c = col0 + wn * TN + j * 16 + hi * 4;
        OutT *o = C + (int64_t)r * P.ldc + c;
        if (whole && c + 4 <= N) {
          store_c4<OutT>(o, acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
        } else {
#pragma unroll
          for (int m = 0; m < 4; m++)
            if (c + m < N) store_c<OutT>(o + m, acc[i][j][m]);
        }
      }
    }
  };
  if (P.c_f32) store(reinterpret_cast<float *>(P.C));
  else store(reinterpret_cast<bf16_t *>(P.C));
}

// ---- bf16, large tiles: two wave groups in turns -------------------------------------------------
// What bounds it: the chip's power.  At full matrix load on real (toggling) data the clock drops
// to ~1.7 GHz, so what counts is energy per product and a matrix pipe that never idles.
//  - MFMA 16x16x32 instead of 32x32x16: same rate per cycle, but a product moves a fifth less
//    operand and accumulator data through the registers (4 KB against 5 KB per 16 kFLOP), and the
//    clock settles higher: 526 -> 461 us on 4096 x 4096 x 22272, 575 -> 530 us on
//    4096 x 22016 x 4096 with everything else equal (1.42 -> 1.62 and 1.28 -> 1.39 PFLOP/s).
//    Consecutive MFMAs share one operand (serpentine order; the other order costs 2 %).
//  - Eight waves, two per SIMD: waves 0-3 and 4-7 (the upper and lower half of the tile's rows) do
//    the same phases half a phase apart, so that one wave of every SIMD issues MFMAs while the
//    other reads fragments and issues copies.  A barrier ends each half phase.  Against a two-
//    stage ring with the copies in one burst after a barrier: 3-5 % at equal MFMA shape.
//  - A K tile is four phases, one quarter (2 x 2) of the wave's output each; both operand tiles are
//    copied in halves (the rows the first / second quarter pair needs), one half per phase, five
//    halves (80 KB of 128 KB LDS) in flight behind the one being waited for.
//  - The fragment reads of a phase are waited for behind its barrier, by the MFMAs that use them,
//    not in front of it: 518 -> 493 us on 4096 x 4096 x 22272 and 101 -> 88 us on
//    300 x 22016 x 4096 on one box.
// A phase: issue the copies of one half tile, start this phase's fragment reads, wait for the half
// that the NEXT phase reads, barrier, MFMAs, barrier.  The waits are counted: half tiles are
// requested in the order B0 A0 B1 A1 of each K tile, IA or IB instructions per wave.
//  - Read after copy: a wave waits for its own share of a half tile in front of a barrier; the
//    second group does so one half phase after the first, still one barrier before the first
//    group's reads.
//  - Copy after read: the reads of a phase are complete before its closing barrier, and the copies
//    that refill a slot are issued at the earliest two half phases after its last reader's.
// Copies past the last tile repeat the last address into the slot that is free anyway, so that
// the counts stay constant.
// BM = 192 is for row counts that need no more tiles of 192 than of 256 (a quarter less padding).
// The last K tile of a segment may be ragged (K % 8 == 0): lanes past the end copy zeros.
// Trailing tiles that would fill less than half of a last round of workgroups are cut along K
// into S slices each (plan_tail below); a slice writes its fp32 partial tile to scratch and
// gemm_tail_reduce_kernel adds the slices in order.  Partial tiles are stored through the caches (the
// other outputs stream past them): the reduction reads them back at once, 5-6 us sooner over 50 MB.
struct GemmPlan {
  int nprob, tail_start, ntail, S;
  int start[GEMM_MAX_PROBLEMS];   // first block of problem p's whole tiles
  int whole[GEMM_MAX_PROBLEMS];   // number of them: tiles [0, whole) in tile_of_lid's order
  int tail0[GEMM_MAX_PROBLEMS];   // first split tile of problem p among all split tiles
  float *part;                    // [S][ntail][BM][256]
};
__device__ __align__(16) const unsigned char gemm_zero16[16] = {};   // source of ragged-K zeros

__device__ __forceinline__ void dma16_at(const void *p, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
               :
               : "v"(p), "s"(lds_addr)
               : "memory", "m0");
}

// problem and tile of split tile tt
__device__ __forceinline__ int tail_tile(const GemmPlan &plan, int tt, int &lid) {
  int pi = 0;
  while (pi + 1 < plan.nprob && plan.tail0[pi + 1] <= tt) pi++;
  lid = plan.whole[pi] + tt - plan.tail0[pi];
  return pi;
}

constexpr int PP_BN = 256, PP_BK = 64;
constexpr size_t pp_lds_bytes(int BM) { return (size_t)2 * (BM + PP_BN) * PP_BK * sizeof(bf16_t); }

template <int BM>
__global__ __launch_bounds__(512) void gemm_bf16_pp_kernel(GemmBatch args, GemmPlan plan) {
  constexpr int BN = PP_BN, BK = PP_BK, ROWB = BK * 2;
  constexpr int HA = BM / 2 * ROWB, HB = BN / 2 * ROWB, STAGE = 2 * (HA + HB);   // half tiles in bytes
  constexpr int HM = BM / 4, MH = HM / 16, NH = 2;   // a wave's rows / 16-row blocks per half
  constexpr int PA = BM / 16, PB = BN / 16;          // 1 KiB pieces of a half tile
  constexpr int IA = (PA + 7) / 8, IB = (PB + 7) / 8;
  static_assert(BM % 64 == 0 && PB % 8 == 0, "tile shape");

  extern __shared__ __align__(16) unsigned char smem[];
  const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char *)smem;

  // block -> problem, tile and K slice
  int bid = blockIdx.x, pi = 0, lid, slice = 0, S = 1, tt = 0;
  if (bid < plan.tail_start) {
    while (pi + 1 < plan.nprob && plan.start[pi + 1] <= bid) pi++;
    lid = xcd_order(bid - plan.start[pi], plan.whole[pi]);
  } else {
    S = plan.S;
    const int l = xcd_order(bid - plan.tail_start, plan.ntail * S);
    slice = l / plan.ntail;
    tt = l - slice * plan.ntail;
    pi = tail_tile(plan, tt, lid);
  }
  const GemmProblem &P = args.p[pi];
  const int M = P.M, N = P.N;
  int tm, tn;
  tile_of_lid(lid, (M + BM - 1) / BM, (N + BN - 1) / BN, tm, tn);
  const int row0 = tm * BM, col0 = tn * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;

  f32x4_t acc[2 * MH][2 * NH];
#pragma unroll
  for (int i = 0; i < 2 * MH; i++)
#pragma unroll
    for (int j = 0; j < 2 * NH; j++) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  // --- producer side ----------------------------------------------------------------------
  int all_tiles = 0;
  for (int sgi = 0; sgi < P.nseg; sgi++) all_tiles += (P.seg[sgi].K + BK - 1) / BK;
  const int t_first = (int)((int64_t)all_tiles * slice / S);
  const int total = (int)((int64_t)all_tiles * (slice + 1) / S) - t_first;
  const int lrow = lane >> 3, lpos = lane & 7;
  // piece j of this wave; with PA = 12 pieces the last four waves repeat other waves' pieces
  auto piece = [&](int j, int pieces) { return wave + 8 * j < pieces ? wave + 8 * j : 8 * j + (wave & 3); };
  uint32_t offA[2][IA], offB[2][IB];
  const unsigned char *baseA = nullptr, *baseB = nullptr;
  int seg = 0, k0, Kcur = 0, valid = 8;   // valid: 16-byte chunks of a row inside K
  auto setup = [&]() {
    const GemmSeg &Sg = P.seg[seg];
#pragma unroll
    for (int h = 0; h < 2; h++) {
#pragma unroll
      for (int j = 0; j < IA; j++) {
        const int q = piece(j, PA) * 8 + lrow;               // row of the half tile
        int r = row0 + (q / HM) * (BM / 2) + h * HM + q % HM;
        r = r < M ? r : M - 1;
        offA[h][j] = (uint32_t)r * (uint32_t)Sg.lda * 2u + (lpos ^ ((q >> 1) & 7)) * 16;
      }
#pragma unroll
      for (int j = 0; j < IB; j++) {
        const int q = piece(j, PB) * 8 + lrow;
        int c = col0 + (q >> 5) * 64 + h * 32 + (q & 31);
        c = c < N ? c : N - 1;
        offB[h][j] = (uint32_t)c * (uint32_t)Sg.ldb * 2u + (lpos ^ ((q >> 1) & 7)) * 16;
      }
    }
    baseA = reinterpret_cast<const unsigned char *>(Sg.A);
    baseB = reinterpret_cast<const unsigned char *>(Sg.B);
    Kcur = Sg.K;
  };
  {
    int skip = t_first;
    for (;;) {
      const int kt = (P.seg[seg].K + BK - 1) / BK;
      if (skip < kt) break;
      skip -= kt;
      seg++;
    }
    k0 = skip * BK;
  }
  setup();
  const void *ga, *gb;
  auto point = [&]() {
    ga = uniform_ptr(baseA + (size_t)k0 * 2);
    gb = uniform_ptr(baseB + (size_t)k0 * 2);
    valid = Kcur - k0 >= BK ? 8 : (Kcur - k0) >> 3;
  };
  point();
  int issued = 0;   // the tile the producer points at
  auto advance = [&]() {
    issued++;
    if (issued < total) {
      k0 += BK;
      if (k0 >= Kcur) {
        seg++;
        k0 = 0;
        setup();
      }
      point();
    }
  };
  auto issue = [&](const uint32_t *off, const void *base, int n, int pieces, uint32_t l) {
    if (valid == 8) {
#pragma unroll
      for (int j = 0; j < n; j++) dma16(off[j], base, l + piece(j, pieces) * 1024);
    } else {
#pragma unroll
      for (int j = 0; j < n; j++) {
        const int q = piece(j, pieces) * 8 + lrow;
        const unsigned char *p = reinterpret_cast<const unsigned char *>(base) + off[j];
        dma16_at((lpos ^ ((q >> 1) & 7)) < valid ? p : gemm_zero16, l + piece(j, pieces) * 1024);
      }
    }
  };
  auto issueA = [&](int h) { issue(offA[h], ga, IA, PA, lds0 + (issued & 1) * STAGE + h * HA); };
  auto issueB = [&](int h) { issue(offB[h], gb, IB, PB, lds0 + (issued & 1) * STAGE + 2 * HA + h * HB); };

  // --- consumer side ----------------------------------------------------------------------
  const int l15 = lane & 15, hi = lane >> 4;
  const int koff[2] = {(hi ^ (l15 >> 1)) * 16, ((4 + hi) ^ (l15 >> 1)) * 16};   // swizzled chunks
  const unsigned char *a_rd = smem + (wm * HM + l15) * ROWB;
  const unsigned char *b_rd = smem + 2 * HA + (wn * 32 + l15) * ROWB;
  bf16x8_t fa[2][MH], fb0[2][NH], fb1[2][NH];
  auto readA = [&](int st, int h) {
    const unsigned char *p = a_rd + st * STAGE + h * HA;
#pragma unroll
    for (int ks = 0; ks < 2; ks++)
#pragma unroll
      for (int i = 0; i < MH; i++)
        fa[ks][i] = *reinterpret_cast<const bf16x8_t *>(p + i * 16 * ROWB + koff[ks]);
  };
  auto readB = [&](int st, int h, bf16x8_t (&fb)[2][NH]) {
    const unsigned char *p = b_rd + st * STAGE + h * HB;
#pragma unroll
    for (int ks = 0; ks < 2; ks++)
#pragma unroll
      for (int j = 0; j < NH; j++)
        fb[ks][j] = *reinterpret_cast<const bf16x8_t *>(p + j * 16 * ROWB + koff[ks]);
  };
  auto barrier = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  auto mfmas = [&](int h, int j, const bf16x8_t (&fb)[2][NH]) {
#pragma unroll
    for (int ks = 0; ks < 2; ks++)
#pragma unroll
      for (int i = 0; i < MH; i++)
#pragma unroll
        for (int q = 0; q < NH; q++) {
          const int jj = q ^ (i & 1);
          acc[h * MH + i][j * NH + jj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              fb[ks][jj], fa[ks][i], acc[h * MH + i][j * NH + jj], 0, 0, 0);
        }
    // every fragment read of the phase is complete before its closing barrier (those the MFMAs did
    // not need as well: B0 of the next tile)
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  };

  issueB(0); issueA(0); issueB(1); issueA(1);
  advance();
  issueB(0); issueA(0); issueB(1);
  wait_vmcnt<2 * IA + 3 * IB>();     // B0 and A0 of tile 0
  barrier();
  if (wm == 1) barrier();            // the second group runs half a phase behind the first
  readB(0, 0, fb0);
  for (int t = 0; t < total; t++) {
    const int st = t & 1;
    issueA(1);                       // A1(t+1)
    readA(st, 0);
    wait_vmcnt<3 * IA + 2 * IB>();   // B1(t)
    barrier();
    mfmas(0, 0, fb0);
    barrier();
    advance();
    issueB(0);                       // B0(t+2)
    readB(st, 1, fb1);
    wait_vmcnt<2 * IA + 3 * IB>();   // A1(t)
    barrier();
    mfmas(0, 1, fb1);
    barrier();
    issueA(0);                       // A0(t+2)
    readA(st, 1);
    wait_vmcnt<3 * IA + 2 * IB>();   // B0(t+1)
    barrier();
    mfmas(1, 0, fb0);
    barrier();
    issueB(1);                       // B1(t+2)
    readB(st ^ 1, 0, fb0);           // B0(t+1)
    wait_vmcnt<2 * IA + 3 * IB>();   // A0(t+1)
    barrier();
    mfmas(1, 1, fb1);
    barrier();
  }
  wait_vmcnt<0>();                   // the copies issued past the end have to be out of the ring
  if (wm == 0) barrier();

  // --- epilogue: through per-wave LDS tiles of 32 rows x 64 columns, so that every global store is
  // 16 bytes per lane and whole 128-byte (or longer) row segments; streaming stores, an output
  // tile is never read again by this launch
  __syncthreads();
  auto store_rows = [&](auto *C, int64_t ldc, int r0, int c0, int rows, int cols, bool streaming) {
    typedef typename std::remove_pointer<decltype(C)>::type OutT;
    constexpr int PER = 16 / (int)sizeof(OutT), TN = 64, EP = TN + PER;
    constexpr int CPW = TN / PER, RPW = 64 / CPW;
    static_assert(8 * 32 * EP * sizeof(OutT) <= pp_lds_bytes(BM), "epilogue tiles fit");
    typedef OutT out4_t __attribute__((ext_vector_type(4)));
    typedef OutT outp_t __attribute__((ext_vector_type(PER)));
    OutT *tile = reinterpret_cast<OutT *>(smem) + wave * 32 * EP;
    const int rr = lane / CPW, cc = lane % CPW;
    const int c = c0 + wn * TN + cc * PER;
#pragma unroll
    for (int i = 0; i < MH; i++) {
#pragma unroll
      for (int ii = 0; ii < 2; ii++)
#pragma unroll
        for (int j = 0; j < 2 * NH; j++) {
          out4_t v;
#pragma unroll
          for (int m = 0; m < 4; m++) v[m] = (OutT)acc[i * 2 + ii][j][m];
          *reinterpret_cast<out4_t *>(tile + (ii * 16 + l15) * EP + j * 16 + hi * 4) = v;
        }
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int p = 0; p < 32 / RPW; p++) {
        const int rl = p * RPW + rr;
        const int r = r0 + wm * (BM / 2) + i * 32 + rl;
        const outp_t v = *reinterpret_cast<const outp_t *>(tile + rl * EP + cc * PER);
        if (r < rows && c < cols) {
          if (streaming) __builtin_nontemporal_store(v, reinterpret_cast<outp_t *>(C + r * ldc + c));
          else *reinterpret_cast<outp_t *>(C + r * ldc + c) = v;
        }
      }
      __builtin_amdgcn_wave_barrier();
    }
  };
  if (S > 1) {
    store_rows(plan.part + ((int64_t)slice * plan.ntail + tt) * (BM * BN), BN, 0, 0, BM, BN, false);
    return;
  }
  const int per = P.c_f32 ? 4 : 8;
  if ((N % per) == 0 && (P.ldc % per) == 0 && (reinterpret_cast<uintptr_t>(P.C) & 15) == 0) {
    if (P.c_f32) store_rows(reinterpret_cast<float *>(P.C), P.ldc, row0, col0, M, N, true);
    else store_rows(reinterpret_cast<bf16_t *>(P.C), P.ldc, row0, col0, M, N, true);
    return;
  }
  // outputs whose rows are not whole 16-byte pieces (an odd number of experts, say)
#pragma unroll
  for (int i = 0; i < 2 * MH; i++) {
    const int r = row0 + wm * (BM / 2) + i * 16 + l15;
    if (r >= M) continue;
#pragma unroll
    for (int j = 0; j < 2 * NH; j++)
#pragma unroll
      for (int m = 0; m < 4; m++) {
        const int c = col0 + wn * 64 + j * 16 + hi * 4 + m;
        if (c >= N) continue;
        if (P.c_f32) store_c<float>(reinterpret_cast<float *>(P.C) + r * P.ldc + c, acc[i][j][m]);
        else store_c<bf16_t>(reinterpret_cast<bf16_t *>(P.C) + r * P.ldc + c, acc[i][j][m]);
      }
  }
}

// Adds the S partial tiles of every split tile in slice order and writes them out.  Bound by the
// partials' latency and rate: a thread owns 4 columns of a row (4 rows per workgroup), and requests
// up to 8 slices before it adds the first.
template <int BM>
__global__ __launch_bounds__(256) void gemm_tail_reduce_kernel(GemmBatch args, GemmPlan plan) {
  constexpr int BN = PP_BN, INFLIGHT = 8;
  const int tt = blockIdx.x;
  int lid;
  const GemmProblem &P = args.p[tail_tile(plan, tt, lid)];
  int tm, tn;
  tile_of_lid(lid, (P.M + BM - 1) / BM, (P.N + BN - 1) / BN, tm, tn);
  const int rt = blockIdx.y * 4 + (threadIdx.x >> 6), ct = (threadIdx.x & 63) * 4;
  const int r = tm * BM + rt, c = tn * BN + ct;
  if (r >= P.M || c >= P.N) return;
  const float *src = plan.part + (int64_t)tt * (BM * BN) + rt * BN + ct;
  const int64_t step = (int64_t)plan.ntail * (BM * BN);
  f32x4_t a = {0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < plan.S; s0 += INFLIGHT) {
    f32x4_t v[INFLIGHT];
#pragma unroll
    for (int i = 0; i < INFLIGHT; i++)   // (a slice past the last one is read again and not added)
      v[i] = *reinterpret_cast<const f32x4_t *>(src + (s0 + i < plan.S ? s0 + i : s0) * step);
#pragma unroll
    for (int i = 0; i < INFLIGHT; i++)
      if (s0 + i < plan.S) a += v[i];
  }
  if (c + 4 <= P.N && (P.ldc & 3) == 0 && (reinterpret_cast<uintptr_t>(P.C) & 15) == 0) {
    if (P.c_f32) store_c4<float>(reinterpret_cast<float *>(P.C) + r * P.ldc + c, a[0], a[1], a[2], a[3]);
    else store_c4<bf16_t>(reinterpret_cast<bf16_t *>(P.C) + r * P.ldc + c, a[0], a[1], a[2], a[3]);
    return;
  }
  for (int i = 0; i < 4 && c + i < P.N; i++) {
    if (P.c_f32) reinterpret_cast<float *>(P.C)[r * P.ldc + c + i] = a[i];
    else reinterpret_cast<bf16_t *>(P.C)[r * P.ldc + c + i] = (bf16_t)a[i];
  }
}

// ---- bf16, one to four rows (decode) ---------------------------------------------------------------
// Matrix-vector products: bound by streaming the weights once.  A wavefront takes RN rows of B (output
// columns), its lanes 16-byte pieces of the same 1 KiB run of each, UN runs requested while the UN
// before them are used (two register sets; streaming loads: without the hint 76 against 70.5 us per
// token of the 7B block).  The rows of A wait in LDS.  No matrix instruction: a row tile would be
// padding but for one to four rows, and products of few columns would have to be cut along K into
// launches of their own.  Lane sums are fp32, added by a butterfly.
// One token of the 7B block: gate/up 39 -> 31 us (5.8 TB/s), down 21 + 4 -> 18 us.
constexpr int GEMV_MAX_ROWS = 4;
constexpr int GEMV_WAVES = 8;

template <int MR, int RN, int UN, bool RANK>
__global__ __launch_bounds__(GEMV_WAVES * 64) void gemm_bf16_rows_kernel(GemmBatch args, FewRank rk) {
  extern __shared__ __align__(16) unsigned char smem[];
  bf16_t *xs = reinterpret_cast<bf16_t *>(smem);       // [MR][segments of K one after the other]
  const GemmProblem &P = args.p[blockIdx.z];
  const int N = P.N;
  if ((int)blockIdx.x * GEMV_WAVES * RN >= N) return;   // problems of one launch may differ in N
  int Ksum = 0;
  for (int sgi = 0; sgi < P.nseg; sgi++) Ksum += P.seg[sgi].K;
  {
    int at = 0;
    for (int sgi = 0; sgi < P.nseg; sgi++) {
      const GemmSeg &S = P.seg[sgi];
#pragma unroll
      for (int m = 0; m < MR; m++) {
        const bf16_t *a = reinterpret_cast<const bf16_t *>(S.A) + (int64_t)(m < P.M ? m : 0) * S.lda;
        for (int c = threadIdx.x * 8; c < S.K; c += GEMV_WAVES * 64 * 8)
          *reinterpret_cast<bf16x8_t *>(xs + m * Ksum + at + c) = *reinterpret_cast<const bf16x8_t *>(a + c);
      }
      at += S.K;
    }
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n0 = (blockIdx.x * GEMV_WAVES + wave) * RN;
  // the rank term: lane j r + q holds B_down[e_j][n][q]; its factor s w_j Q_j[q] is summed into LDS meanwhile
  float bd[RN][MR];
  float *sq = reinterpret_cast<float *>(xs + (size_t)MR * Ksum);
  if constexpr (RANK) {
    const int v = lane < rk.k * rk.r ? lane : 0;
#pragma unroll
    for (int m = 0; m < MR; m++) {
      const int e = rk.idx[(m < P.M ? m : 0) * rk.k + v / rk.r];
#pragma unroll
      for (int i = 0; i < RN; i++)
        bd[i][m] = (float)rk.B_down[((int64_t)e * N + (n0 + i < N ? n0 + i : N - 1)) * rk.r + v % rk.r];
    }
    for (int m = 0; m < P.M; m++)
      few_rank_sums(rk, m, blockIdx.x == 0, GEMV_WAVES * 64, sq + MR * 64, sq + m * 64);
  }
  float acc[RN][MR];
#pragma unroll
  for (int i = 0; i < RN; i++)
#pragma unroll
    for (int m = 0; m < MR; m++) acc[i][m] = 0.f;
  __syncthreads();
  if (n0 >= N) return;
  int at = 0;
  for (int sgi = 0; sgi < P.nseg; sgi++) {
    const GemmSeg &S = P.seg[sgi];
    const bf16_t *b[RN];
#pragma unroll
    for (int i = 0; i < RN; i++)
      b[i] = reinterpret_cast<const bf16_t *>(S.B) + (int64_t)(n0 + i < N ? n0 + i : N - 1) * S.ldb;
    auto add = [&](const bf16x8_t (&w)[RN], int k) {
#pragma unroll
      for (int m = 0; m < MR; m++) {
        const bf16x8_t x = *reinterpret_cast<const bf16x8_t *>(xs + m * Ksum + at + k);
#pragma unroll
        for (int i = 0; i < RN; i++)
#pragma unroll
          for (int e = 0; e < 8; e++) acc[i][m] = fmaf((float)w[i][e], (float)x[e], acc[i][m]);
      }
    };
    int k0 = lane * 8;
    const int whole = S.K / (512 * UN);
    bf16x8_t w[2][UN][RN];
    auto load = [&](int buf, int k) {
#pragma unroll
      for (int u = 0; u < UN; u++)
#pragma unroll
        for (int i = 0; i < RN; i++)
          w[buf][u][i] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8_t *>(b[i] + k + u * 512));
    };
    if (whole > 0) load(0, k0);
    for (int it = 0; it < whole; it += 2) {   // two register sets: the next runs are on their way
#pragma unroll
      for (int h = 0; h < 2; h++) {
        if (it + h < whole) {
          if (it + h + 1 < whole) load(h ^ 1, k0 + 512 * UN);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int u = 0; u < UN; u++) add(w[h][u], k0 + u * 512);
          k0 += 512 * UN;
        }
      }
    }
    for (; k0 < S.K; k0 += 512) {
      bf16x8_t v[RN];
#pragma unroll
      for (int i = 0; i < RN; i++) v[i] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8_t *>(b[i] + k0));
      add(v, k0);
    }
    at += S.K;
  }
  if constexpr (RANK) {
    if (lane < rk.k * rk.r) {
#pragma unroll
      for (int i = 0; i < RN; i++)
#pragma unroll
        for (int m = 0; m < MR; m++) acc[i][m] = fmaf(sq[(m < P.M ? m : 0) * 64 + lane], bd[i][m], acc[i][m]);
    }
  }
#pragma unroll
  for (int i = 0; i < RN; i++)
#pragma unroll
    for (int m = 0; m < MR; m++) {
      float v = acc[i][m];
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
      if (lane == 0 && n0 + i < N && m < P.M) {
        if (P.c_f32) reinterpret_cast<float *>(P.C)[m * P.ldc + n0 + i] = v;
        else reinterpret_cast<bf16_t *>(P.C)[m * P.ldc + n0 + i] = (bf16_t)v;
      }
    }
}

// ---- fp32 storage ---------------------------------------------------------------------------
// MFMA 16x16x4 fp32 (each product and sum rounded to fp32) on a TB x TB tile; the waves of a
// workgroup take every NWV-th 16-wide run of K (of all segments in a row) and their sums are added
// in wave order through LDS.  Fragments come straight from memory as 16-byte loads: lane (l15, hi)
// holds elements 4 hi .. 4 hi + 3 of a row's run, i.e. four MFMA steps whose K order is permuted
// alike on both sides.  fp32 problems here are small (the configuration the numerics are checked
// on: 256 x 344 x 128 and the like), so what bounds them is the latency of a chain of loads: eight
// waves on a 32 x 32 tile walk K in an eighth of the steps and cover the chip with tiles, where a
// 64 x 64 tile staged through LDS left most of it idle (256 x 128 x 824: 64 -> 11 us).  Where 64 x 64
// tiles are many enough for every CU, they halve the loads per product.
//
// A problem marked by_rows takes a wave per row and two columns instead: lane l sums the 8-wide pieces l, l + 64, .. of the
// row, a butterfly adds the lanes.  Its chains are K / 64 long, not K / 8: the routing weights, which exponentiate
// these sums, are 1.2e-7 from 64 bits at K = 4096, and 3.1e-7 on the tiles.
__device__ __forceinline__ void f32_rows(const GemmProblem &P, int first, int step) {
  constexpr int NC = 2;   // columns of an item (with four the kernel's registers cost a workgroup per CU)
  const int lane = threadIdx.x & 63, groups = (P.N + NC - 1) / NC;
  const GemmSeg &S = P.seg[0];
  for (int64_t item = first; item < (int64_t)P.M * groups; item += step) {
    const int64_t row = item / groups;
    const int n0 = (int)(item - row * groups) * NC;
    const float *a = reinterpret_cast<const float *>(S.A) + row * S.lda;
    float acc[NC];
#pragma unroll
    for (int n = 0; n < NC; n++) acc[n] = 0.f;
    for (int c = lane * 8; c < S.K; c += 64 * 8) {   // K % 8 == 0
      Vec8<float> av;
      av.load(a + c);
#pragma unroll
      for (int n = 0; n < NC; n++) {
        Vec8<float> bv;
        bv.load(reinterpret_cast<const float *>(S.B) + (int64_t)(n0 + n < P.N ? n0 + n : P.N - 1) * S.ldb + c);
#pragma unroll
        for (int i = 0; i < 8; i++) acc[n] = fmaf(av.get(i), bv.get(i), acc[n]);
      }
    }
#pragma unroll
    for (int n = 0; n < NC; n++) {
      float v = acc[n];
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
      if (lane == n && n0 + n < P.N) reinterpret_cast<float *>(P.C)[row * P.ldc + n0 + n] = v;
    }
  }
}

__global__ __launch_bounds__(256) void f32_rows_kernel(GemmBatch args) {
  f32_rows(args.p[0], blockIdx.x * 4 + (threadIdx.x >> 6), gridDim.x * 4);
}

// ROWS: the launch has such a problem (an instance of its own: the branch changes the compiler's schedule of
// the tiles, a tenth more time where 64 x 64 tiles cover the chip, which therefore have the rows in a launch
// behind them)
template <int TB, int NWV, bool ROWS>
__global__ __launch_bounds__(NWV * 64) void gemm_f32_kernel(GemmBatch args) {
  constexpr int NB = TB / 16;
  __shared__ float red[NWV][TB][TB + (TB == 64 ? 0 : 4)];   // 64 KB at most
  const GemmProblem &P = args.p[blockIdx.z];
  if constexpr (ROWS) {
    if (P.by_rows) {   // workgroup-uniform
      f32_rows(P, blockIdx.x * NWV + (threadIdx.x >> 6), gridDim.x * NWV);
      return;
    }
  }
  const int M = P.M, N = P.N;
  const int tiles_m = (M + TB - 1) / TB, tiles_n = (N + TB - 1) / TB;
  if ((int)blockIdx.x >= tiles_m * tiles_n) return;   // problems of one launch may differ in shape
  const int row0 = blockIdx.x / tiles_n * TB, col0 = blockIdx.x % tiles_n * TB;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l15 = lane & 15, hi = lane >> 4;
  int arow[NB], bcol[NB];
#pragma unroll
  for (int i = 0; i < NB; i++) {   // rows past the edge: the last one again, never stored
    arow[i] = row0 + i * 16 + l15 < M ? row0 + i * 16 + l15 : M - 1;
    bcol[i] = col0 + i * 16 + l15 < N ? col0 + i * 16 + l15 : N - 1;
  }
  f32x4_t acc[NB][NB];
#pragma unroll
  for (int i = 0; i < NB; i++)
#pragma unroll
    for (int j = 0; j < NB; j++) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  int turn = wave;   // runs until this wave's next one
  for (int sgi = 0; sgi < P.nseg; sgi++) {
    const GemmSeg &S = P.seg[sgi];
    const float *A = reinterpret_cast<const float *>(S.A), *B = reinterpret_cast<const float *>(S.B);
    const int runs = (S.K + 15) >> 4;
    const int mine = turn < runs ? (runs - turn + NWV - 1) / NWV : 0;
    for (int it = 0; it < mine; it++) {   // (two runs in flight per wave measured slower: 1200 -> 1660 us
                                          // per step at 2048 x 1024 x 2752, 102 -> 106 at the small one)
      const int k = (turn + it * NWV) * 16 + hi * 4;
      const bool in = k < S.K;   // K % 8 == 0: a lane's four elements are all in or all out
      f32x4_t fa[NB], fb[NB];
#pragma unroll
      for (int i = 0; i < NB; i++) {
        fa[i] = *reinterpret_cast<const f32x4_t *>(A + (int64_t)arow[i] * S.lda + (in ? k : 0));
        fb[i] = *reinterpret_cast<const f32x4_t *>(B + (int64_t)bcol[i] * S.ldb + (in ? k : 0));
      }
      if (!in) {
#pragma unroll
        for (int i = 0; i < NB; i++) fa[i] = fb[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
      for (int m = 0; m < 4; m++)
#pragma unroll
        for (int i = 0; i < NB; i++)
#pragma unroll
          for (int j = 0; j < NB; j++)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[j][m], fa[i][m], acc[i][j], 0, 0, 0);
    }
    turn += mine * NWV - runs;
  }
#pragma unroll
  for (int i = 0; i < NB; i++)
#pragma unroll
    for (int j = 0; j < NB; j++)
      *reinterpret_cast<f32x4_t *>(&red[wave][i * 16 + l15][j * 16 + hi * 4]) = acc[i][j];
  __syncthreads();
  float *C = reinterpret_cast<float *>(P.C);
  const bool vec = (P.ldc & 3) == 0 && (reinterpret_cast<uintptr_t>(C) & 15) == 0;
  for (int x = threadIdx.x; x < TB * TB / 4; x += NWV * 64) {
    const int rl = x / (TB / 4), cl = x % (TB / 4) * 4;
    const int r = row0 + rl, c = col0 + cl;
    if (r >= M || c >= N) continue;
    f32x4_t v = *reinterpret_cast<const f32x4_t *>(&red[0][rl][cl]);
#pragma unroll
    for (int w = 1; w < NWV; w++) v += *reinterpret_cast<const f32x4_t *>(&red[w][rl][cl]);
    if (vec && c + 4 <= N) {
      *reinterpret_cast<f32x4_t *>(C + (int64_t)r * P.ldc + c) = v;
    } else {
      for (int m = 0; m < 4 && c + m < N; m++) C[(int64_t)r * P.ldc + c + m] = v[m];
    }
  }
}

// floating-point operations a launch executes (2 M N K over its problems' K segments)
static double batch_flops(const GemmBatch &b, int nprob) {
  double fl = 0.0;
  for (int i = 0; i < nprob; i++)
    for (int sgi = 0; sgi < b.p[i].nseg; sgi++)
      fl += 2.0 * b.p[i].M * (double)b.p[i].N * b.p[i].seg[sgi].K;
  return fl;
}

// launches that carry a frozen projection (more than 128 output columns) count as GEMM launches for the
// measurement hook; a launch of narrow rank-r or router problems does not
static int batch_kind(const GemmBatch &b, int nprob) {
  for (int i = 0; i < nprob; i++)
    if (b.p[i].N > 128) return PROF_GEMM;
  return PROF_OTHER;
}
static void mark_end(int slot, const GemmBatch &b, int nprob, hipStream_t st) {
  if (slot >= 0) prof_mark_end(slot, st, batch_kind(b, nprob) == PROF_GEMM ? batch_flops(b, nprob) : 0.0);
}

template <int BM, int BN, int BK, int WGM, int WGN, typename OutT>
static hipError_t launch_bf16(const GemmBatch &b, int nprob, hipStream_t st) {
  constexpr size_t smem = (size_t)2 * (BM + BN) * (BK + 8) * sizeof(bf16_t);
  auto kern = gemm_bf16_kernel<BM, BN, BK, WGM, WGN, OutT>;
  static bool attr_set = false;   // per template instance; the attribute is per function
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  const int tiles = ((b.p[0].M + BM - 1) / BM) * ((b.p[0].N + BN - 1) / BN);
  const int slot = prof_on() ? prof_mark_begin(batch_kind(b, nprob), st) : -1;
  hipLaunchKernelGGL(kern, dim3(tiles, 1, nprob), dim3(WGM * WGN * 64), smem, st, b);
  mark_end(slot, b, nprob, st);
  return hipGetLastError();
}

// bytes of a launch's B operands
static double b_bytes(const GemmBatch &b, int nprob) {
  double by = 0.0;
  for (int i = 0; i < nprob; i++)
    for (int sgi = 0; sgi < b.p[i].nseg; sgi++) by += 2.0 * b.p[i].N * b.p[i].seg[sgi].K;
  return by;
}
constexpr double STREAM_BYTES = 64.0 * 1024 * 1024;

template <int BM, int BN, int STAGES>
static hipError_t launch_few(const GemmBatch &b, int nprob, bool streaming, const FewRank &rk, hipStream_t st) {
  constexpr size_t smem = (size_t)STAGES * (BM + BN) * 128;
  auto kern = gemm_bf16_few_kernel<BM, BN, STAGES>;
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  FewPlan plan{};
  plan.nprob = nprob;
  plan.streaming = streaming;
  int at = 0;
  for (int i = 0; i < nprob; i++) {
    plan.start[i] = at;
    at += (b.p[i].N + BN - 1) / BN;
  }
  const int slot = prof_on() ? prof_mark_begin(batch_kind(b, nprob), st) : -1;
  plan.tiles = at;
  hipLaunchKernelGGL(kern, dim3(at + rk.T), dim3(256), smem, st, b, plan, rk);
  mark_end(slot, b, nprob, st);
  return hipGetLastError();
}

template <int BM>
static hipError_t launch_few_w(const GemmBatch &b, int nprob, int width, bool streaming, const FewRank &rk,
                               hipStream_t st) {
  switch (width) {
    case 32: return launch_few<BM, 32, 4>(b, nprob, streaming, rk, st);
    case 64: return launch_few<BM, 64, 4>(b, nprob, streaming, rk, st);
    case 96: return launch_few<BM, 96, 4>(b, nprob, streaming, rk, st);
    default: return launch_few<BM, 128, 4>(b, nprob, streaming, rk, st);
  }
}
static hipError_t launch_few_m(const GemmBatch &b, int nprob, int width, bool streaming, const FewRank &rk,
                               hipStream_t st) {
  const int M = b.p[0].M;
  if (M <= 32) return launch_few_w<32>(b, nprob, width, streaming, rk, st);
  return M <= 64 ? launch_few_w<64>(b, nprob, width, streaming, rk, st)
                 : launch_few_w<128>(b, nprob, width, streaming, rk, st);
}

// Column width of the tiles of a few-rows launch: the one with the least columns per CU, the widest of
// equals.  Whole forwards, against 64 always: 64 tokens of the 7B block 92.9 -> 84.0 us, 128 of the 13B
// block 157.9 -> 137.0, 128 of a 1024 x 2752 one 41.5 -> 38.6 (32 columns; 41.0 with 64 at least).
static int few_width(const GemmBatch &b, int nprob) {
  int best = 64, cost = 1 << 30;
  const int widths[4] = {128, 96, 64, 32};
  for (int w : widths) {
    int tiles = 0;
    for (int i = 0; i < nprob; i++) tiles += (b.p[i].N + w - 1) / w;
    const int c = (tiles + 255) / 256 * w;
    if (c < cost) {
      cost = c;
      best = w;
    }
  }
  return best;
}

// The direct-to-LDS kernels need 32-bit operand offsets, and (the narrow-tile one) whole K tiles.
static bool dl_eligible(const GemmBatch &b, int nprob, int BK) {
  for (int i = 0; i < nprob; i++) {
    const GemmProblem &p = b.p[i];
    for (int sgi = 0; sgi < p.nseg; sgi++) {
      const GemmSeg &sg = p.seg[sgi];
      if (sg.K <= 0 || sg.K % BK) return false;
      if ((uint64_t)p.M * (uint64_t)sg.lda * 2 >= (1ull << 32)) return false;
      if ((uint64_t)p.N * (uint64_t)sg.ldb * 2 >= (1ull << 32)) return false;
    }
  }
  return true;
}

// How many trailing tiles of a launch of `tiles` to cut along K, and into how many slices.  The
// last round of workgroups (one per CU) takes as long as a full one however few tiles it holds;
// with S slices per tile it takes 1/S of that, plus the partial tiles' way through memory.
// Per K tile a tile needs ~1.2 us (1.3 with few CUs at work, 1.5 with all of them and less clock),
// partial tiles are written and read at ~6 TB/s, and the second launch costs ~5 us.  Measured
// (us, uncut / cut, operands in HBM): 300 x 4096 x 11136 209 / 62 (7 slices), 300 x 11008 x 4096
// 88 / 68 (2), 517 x 22016 x 4096 171 / 113 (2 of 258 tiles in 16), 1999 x 4096 x 22272 425 / 277 (2),
// 236 x 1024 x 4096 85 / 23 (12).
static void plan_tail(int tiles, int ktiles, int BM, size_t part_floats, int &ntail, int &S) {
  constexpr int CUS = 256;
  ntail = 0;
  S = 1;
  const int tail = tiles % CUS;
  if (tail == 0 || tail > CUS / 2) return;
  const double tile_mb = BM * PP_BN * 8e-6;   // MB written and read again per partial tile
  double best = 0.0;
  for (int n = 2; n <= 32 && n * tail <= CUS && ktiles / n >= 4 && (size_t)n * tail * BM * PP_BN <= part_floats; n++) {
    const double gain = 1.2 * ktiles * (1.0 - 1.0 / n) - (tail * n * tile_mb / 6.0 + 5.0);
    if (gain > best) {
      best = gain;
      ntail = tail;
      S = n;
    }
  }
}

static int pp_tiles(const GemmProblem &p, int BM) {
  return ((p.M + BM - 1) / BM) * ((p.N + PP_BN - 1) / PP_BN);
}

template <int BM>
static hipError_t launch_pp(const GemmBatch &b, int nprob, int ntail, int S, float *part, hipStream_t st) {
  constexpr size_t smem = pp_lds_bytes(BM);
  auto kern = gemm_bf16_pp_kernel<BM>;
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  GemmPlan plan{};
  plan.nprob = nprob;
  plan.ntail = ntail;
  plan.S = S;
  plan.part = part;
  int total = 0, at = 0, before = 0;
  for (int i = 0; i < nprob; i++) total += pp_tiles(b.p[i], BM);
  const int whole_all = total - ntail;
  for (int i = 0; i < GEMM_MAX_PROBLEMS; i++) {
    const int n = i < nprob ? pp_tiles(b.p[i], BM) : 0;
    int w = whole_all - before;                  // whole tiles left for this problem
    w = w < 0 ? 0 : (w > n ? n : w);
    plan.start[i] = at;
    plan.whole[i] = w;
    plan.tail0[i] = before + w - whole_all;      // <= 0 up to the first problem with split tiles
    if (plan.tail0[i] < 0) plan.tail0[i] = 0;
    at += w;   // no padding between problems: 256 tiles are 32 per XCD, one round
    before += n;
  }
  plan.tail_start = at;
  // (a cut launch and the one that adds its slices count as one)
  const int slot = prof_on() ? prof_mark_begin(batch_kind(b, nprob), st) : -1;
  hipLaunchKernelGGL(kern, dim3(at + ntail * S), dim3(512), smem, st, b, plan);
  if (ntail > 0) hipLaunchKernelGGL(gemm_tail_reduce_kernel<BM>, dim3(ntail, BM / 4), dim3(256), 0, st, b, plan);
  mark_end(slot, b, nprob, st);
  return hipGetLastError();
}

// Large-tile launch of any number of problems (row counts may differ); only >= 0: of that one alone, its
// tiles being cut as in the launch of all.
static hipError_t launch_large(const GemmBatch &b, int nprob, const GemmScratch &scratch, hipStream_t st,
                               int only = -1) {
  // 192 rows per tile where that needs no more tiles than 256 (129-192, 257-384, 513-576 rows)
  bool m192 = true;
  int ktiles = 1 << 30;
  for (int i = 0; i < nprob; i++) {
    if ((b.p[i].M + 191) / 192 != (b.p[i].M + 255) / 256) m192 = false;
    int kt = 0;
    for (int sgi = 0; sgi < b.p[i].nseg; sgi++) kt += (b.p[i].seg[sgi].K + PP_BK - 1) / PP_BK;
    ktiles = kt < ktiles ? kt : ktiles;
  }
  const int BM = m192 ? 192 : 256;
  int tiles = 0, ntail, S;
  for (int i = 0; i < nprob; i++) tiles += pp_tiles(b.p[i], BM);
  plan_tail(tiles, ktiles, BM, scratch.part ? scratch.floats : 0, ntail, S);
  if (only >= 0) {
    int behind = 0;   // tiles of the problems that follow: the trailing ones are cut first
    for (int i = only + 1; i < nprob; i++) behind += pp_tiles(b.p[i], BM);
    const int own = pp_tiles(b.p[only], BM);
    ntail = ntail <= behind ? 0 : ntail - behind < own ? ntail - behind : own;
    GemmBatch one;
    for (int i = 0; i < GEMM_MAX_PROBLEMS; i++) one.p[i] = b.p[only];
    return m192 ? launch_pp<192>(one, 1, ntail, S, scratch.part, st)
                : launch_pp<256>(one, 1, ntail, S, scratch.part, st);
  }
  return m192 ? launch_pp<192>(b, nprob, ntail, S, scratch.part, st)
              : launch_pp<256>(b, nprob, ntail, S, scratch.part, st);
}

// Two rows of B per wave, one where the columns are so few that two would leave SIMDs empty.  One token of
// the 7B block: four rows per wave 73.7 us, two 71.6, and with one for the down projection's 4096 columns
// 70.5 against 71.4; one row through a 4096 x 4096 linear layer 13.8 -> 12.7.
static hipError_t launch_rows(const GemmBatch &b, int nprob, hipStream_t st) {
  int n = 0, total = 0, kmax = 0;
  for (int i = 0; i < nprob; i++) {
    n = b.p[i].N > n ? b.p[i].N : n;
    total += b.p[i].N;
    int kt = 0;
    for (int sgi = 0; sgi < b.p[i].nseg; sgi++) kt += b.p[i].seg[sgi].K;
    kmax = kt > kmax ? kt : kmax;
  }
  // (three and four rows come with at most 8192 columns: one row of B per wave)
  const int M = b.p[0].M, mr = M == 1 ? 1 : M == 2 ? 2 : 4, rn = mr < 4 && total > 8192 ? 2 : 1;
  const size_t smem = (size_t)mr * kmax * sizeof(bf16_t);
  const dim3 grid((n + GEMV_WAVES * rn - 1) / (GEMV_WAVES * rn), 1, nprob), block(GEMV_WAVES * 64);
  const int slot = prof_on() ? prof_mark_begin(batch_kind(b, nprob), st) : -1;
  const FewRank rk{};
  if (mr == 4) hipLaunchKernelGGL((gemm_bf16_rows_kernel<4, 1, 4, false>), grid, block, smem, st, b, rk);
  else if (mr == 2 && rn == 2) hipLaunchKernelGGL((gemm_bf16_rows_kernel<2, 2, 4, false>), grid, block, smem, st, b, rk);
  else if (mr == 2) hipLaunchKernelGGL((gemm_bf16_rows_kernel<2, 1, 4, false>), grid, block, smem, st, b, rk);
  else if (rn == 2) hipLaunchKernelGGL((gemm_bf16_rows_kernel<1, 2, 4, false>), grid, block, smem, st, b, rk);
  else hipLaunchKernelGGL((gemm_bf16_rows_kernel<1, 1, 4, false>), grid, block, smem, st, b, rk);
  mark_end(slot, b, nprob, st);
  return hipGetLastError();
}

// Rows and contraction length for which the row kernel is the better one whatever the columns: one and
// two rows (from three on, reading A out of LDS costs more than the matrix tiles' padding: three rows of
// the 7B block 89 us against 85, four of the 13B block 122 against 108), their copy of A at most 64 KiB of
// LDS.  launch_gemm also takes three and four rows of one or two problems into at most 8192 columns, which
// are too few column tiles (forward of a linear layer of rank 16, 4 rows, 4096 -> 1024: 28 -> 13 us); the
// block's forward launches, of five problems or of one per K slice, are not (3 tokens of 1024 x 2752:
// 38.4 us per pass on the tiles, 43.4 here).
bool gemm_rows_ok(int dtype, int M, int K) {
  return dtype == MIXLORA_BF16 && M >= 1 && M <= 2 && (size_t)M * K * sizeof(bf16_t) <= 65536;
}

bool gemm_few_rank_ok(int dtype, int M, int N, int K) {
  return dtype == MIXLORA_BF16 && M >= 1 && M <= 128 && K % 64 == 0 && (uint64_t)N * K * 2 < (1ull << 32);
}
hipError_t launch_gemm_few_rank(const GemmProblem *probs, int nprob, const FewRank &rk, hipStream_t st) {
  if (nprob < 1 || nprob > GEMM_MAX_PROBLEMS || rk.k * rk.r > FEW_RANK_SUMS) return hipErrorInvalidValue;
  GemmBatch b;
  for (int i = 0; i < GEMM_MAX_PROBLEMS; i++) b.p[i] = probs[i < nprob ? i : 0];
  if (b.p[0].M < 1 || b.p[0].M > 128 || !dl_eligible(b, nprob, 64)) return hipErrorInvalidValue;
  return launch_few_m(b, nprob, few_width(b, nprob), b_bytes(b, nprob) >= STREAM_BYTES, rk, st);
}

// The row kernel with the rank-r term of the down projection (one problem, one K segment).  Every workgroup adds
// up the partial sums of the term's left factor (22 KB per token at the 7B shape) while its weights start:
// 18.6 -> 19.9 us against the term as a K segment, which needs a launch of 4.5 us in front of it.
static size_t rows_rank_smem(int mr, int K) {
  return (size_t)mr * K * sizeof(bf16_t) + ((size_t)mr * 64 + GEMV_WAVES * 64) * sizeof(float);
}
bool gemm_rows_rank_ok(int dtype, int M, int K) {
  return dtype == MIXLORA_BF16 && M >= 1 && M <= 2 && rows_rank_smem(M, K) <= 65536;
}
hipError_t launch_gemm_rows_rank(const GemmProblem &p, const FewRank &rk, hipStream_t st) {
  const int K = p.seg[0].K;
  if (p.nseg != 1 || !gemm_rows_rank_ok(MIXLORA_BF16, p.M, K) || rk.k * rk.r > 64) return hipErrorInvalidValue;
  GemmBatch b;
  for (int i = 0; i < GEMM_MAX_PROBLEMS; i++) b.p[i] = p;
  const int mr = p.M, rn = p.N > 8192 ? 2 : 1;
  const dim3 grid((p.N + GEMV_WAVES * rn - 1) / (GEMV_WAVES * rn)), block(GEMV_WAVES * 64);
  const size_t smem = rows_rank_smem(mr, K);
  const int slot = prof_on() ? prof_mark_begin(batch_kind(b, 1), st) : -1;
  if (mr == 2 && rn == 2) hipLaunchKernelGGL((gemm_bf16_rows_kernel<2, 2, 4, true>), grid, block, smem, st, b, rk);
  else if (mr == 2) hipLaunchKernelGGL((gemm_bf16_rows_kernel<2, 1, 4, true>), grid, block, smem, st, b, rk);
  else if (rn == 2) hipLaunchKernelGGL((gemm_bf16_rows_kernel<1, 2, 4, true>), grid, block, smem, st, b, rk);
  else hipLaunchKernelGGL((gemm_bf16_rows_kernel<1, 1, 4, true>), grid, block, smem, st, b, rk);
  mark_end(slot, b, 1, st);
  return hipGetLastError();
}

bool gemm_mixed_rows_ok(int dtype, const GemmProblem *probs, int nprob) {
  if (dtype != MIXLORA_BF16 || nprob < 1 || nprob > GEMM_MAX_PROBLEMS) return false;
  GemmBatch b;
  bool any_big = false;
  for (int i = 0; i < GEMM_MAX_PROBLEMS; i++) b.p[i] = probs[i < nprob ? i : 0];
  for (int i = 0; i < nprob; i++) {
    if (probs[i].M <= 128 || probs[i].N <= 0) return false;
    if (probs[i].N > 128) any_big = true;
  }
  return any_big && dl_eligible(b, nprob, 8);
}

hipError_t launch_gemm(int dtype, const GemmProblem *probs, int nprob, hipStream_t st,
                       const GemmScratch &scratch, int only) {
  if (nprob < 1 || nprob > GEMM_MAX_PROBLEMS || only >= nprob) return hipErrorInvalidValue;
  GemmBatch b;
  for (int i = 0; i < GEMM_MAX_PROBLEMS; i++) b.p[i] = probs[i < nprob ? i : 0];
  // what is launched; the route is chosen from all problems
  GemmBatch l = b;
  if (only >= 0)
    for (int i = 0; i < GEMM_MAX_PROBLEMS; i++) l.p[i] = probs[only];
  const int nl = only >= 0 ? 1 : nprob;
  if (dtype == MIXLORA_F32) {
    int t32 = 0, t64 = 0, all64 = 0, rows = -1;
    for (int i = 0; i < nprob; i++) {
      if (probs[i].M <= 0 || probs[i].N <= 0) return hipErrorInvalidValue;
      if (probs[i].by_rows) {
        if (rows >= 0 || i + 1 != nprob || only >= 0 || probs[i].nseg != 1) return hipErrorInvalidValue;
        rows = i;
        continue;
      }
      const int a = ((probs[i].M + 31) / 32) * ((probs[i].N + 31) / 32);
      const int c = ((probs[i].M + 63) / 64) * ((probs[i].N + 63) / 64);
      t32 = a > t32 ? a : t32;
      t64 = c > t64 ? c : t64;
      all64 += c;
    }
    if (all64 >= 512 || (rows >= 0 && nprob == 1)) {   // two tiles of 64 x 64 per CU
      if (nl > (rows >= 0))
        hipLaunchKernelGGL((gemm_f32_kernel<64, 4, false>), dim3(t64, 1, nl - (rows >= 0)), dim3(256), 0, st, l);
      if (rows >= 0) {
        l.p[0] = probs[rows];
        const int64_t blocks = ((int64_t)l.p[0].M * ((l.p[0].N + 1) / 2) + 3) / 4;
        hipLaunchKernelGGL(f32_rows_kernel, dim3((unsigned)(blocks < 4096 ? blocks : 4096)), dim3(256), 0, st, l);
      }
    } else if (rows >= 0) {
      hipLaunchKernelGGL((gemm_f32_kernel<32, 8, true>), dim3(t32, 1, nl), dim3(512), 0, st, l);
    } else {
      hipLaunchKernelGGL((gemm_f32_kernel<32, 8, false>), dim3(t32, 1, nl), dim3(512), 0, st, l);
    }
    return hipGetLastError();
  }
  const int M = probs[0].M, N = probs[0].N;
  bool uniform = true, any_big = false, same_m = true;
  for (int i = 0; i < nprob; i++) {
    if (probs[i].M != M) same_m = false;
    if (probs[i].N != N || probs[i].c_f32 != probs[0].c_f32) uniform = false;
    if (probs[i].N > 128) any_big = true;
    if (probs[i].N <= 0) return hipErrorInvalidValue;
  }
  if (!same_m) {
    // problems of different row counts (per-token and per-pair operands) can share a launch of
    // the large-tile kernel only: every tile takes M from its own problem
    if (!gemm_mixed_rows_ok(dtype, probs, nprob)) return hipErrorInvalidValue;
    return launch_large(b, nprob, scratch, st, only);
  }
  if (M <= 0) return hipSuccess;
  if (dtype == MIXLORA_BF16 && M <= GEMV_MAX_ROWS) {
    int64_t kmax = 0;
    for (int i = 0; i < nprob; i++) {
      int64_t kt = 0;
      for (int sgi = 0; sgi < probs[i].nseg; sgi++) kt += probs[i].seg[sgi].K;
      kmax = kt > kmax ? kt : kmax;
    }
    int64_t cols = 0;
    for (int i = 0; i < nprob; i++) cols += probs[i].N;
    if (kmax < (1 << 20) && (gemm_rows_ok(dtype, M, (int)kmax) || (nprob <= 2 && cols <= 8192 && kmax * 8 <= 65536)))
      return launch_rows(l, nl, st);
  }
  // Large tiles.  Problems of one launch may differ in N and output type (narrow ones ride in the
  // slack of the last, partially filled round of workgroups).
  if (dtype == MIXLORA_BF16 && M > 128 && any_big && dl_eligible(b, nprob, 8))
    return launch_large(b, nprob, scratch, st, only);
  // Few rows, and too few 64-column tiles to stream the weights (or ragged K, which the narrow tiles do
  // not take): the large tiles cut along K.  28 x 1024 x 4096 and 100 x 5120 x 5120 with their
  // rank-r term 33 -> 30 and 41 -> 38 us; 30 tokens of a 1296 x 4272 block 181 -> 57.
  if (dtype == MIXLORA_BF16 && M <= 128 && any_big && scratch.part && dl_eligible(b, nprob, 8)) {
    int narrow = 0;
    for (int i = 0; i < nprob; i++) narrow += (probs[i].N + 63) / 64;
    if (narrow < 128 || !dl_eligible(b, nprob, 64)) return launch_large(b, nprob, scratch, st, only);
  }
  if (dtype == MIXLORA_BF16 && M <= 128 && any_big && dl_eligible(b, nprob, 64)) {
    // few rows (decode-shaped calls): the launch is bound by streaming the weights once, so the
    // tiles are narrow enough to cover the chip
    // Weights of 64 MiB or more are streamed past the caches: the last level (256 MiB) would not hold
    // them until the next pass anyway, and reading them costs less without the attempt (64 tokens of
    // the 7B block 91.1 -> 84.0 us, 12 tokens 81.9 -> 75.0).  Smaller ones may still be there
    // (52 MB, with an earlier kernel: 40.6 us cached, 44.4 streamed).
    return launch_few_m(l, nl, few_width(b, nprob), b_bytes(b, nprob) >= STREAM_BYTES, FewRank{}, st);
  }
  if (!uniform || nprob > 2) {   // the generic kernels take uniform batches of at most two
    for (int i = 0; i < nprob; i++) {
      if (only >= 0 && i != only) continue;
      const hipError_t e = launch_gemm(dtype, probs + i, 1, st, scratch);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  const bool f32out = probs[0].c_f32 != 0;
  if (N <= 128 || M <= 128) {
    return f32out ? launch_bf16<128, 128, 64, 2, 2, float>(l, nl, st)
                  : launch_bf16<128, 128, 64, 2, 2, bf16_t>(l, nl, st);
  }
  return f32out ? launch_bf16<256, 256, 64, 2, 4, float>(l, nl, st)
                : launch_bf16<256, 256, 64, 2, 4, bf16_t>(l, nl, st);
}

}  // namespace mixlora
