// Internal declarations shared by the HIP translation units of libmixlora (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/mixlora.h"

namespace mixlora {

typedef __bf16 bf16_t;
typedef bf16_t bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// ---- element access in the storage dtype, arithmetic always in fp32 -------------------
__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(bf16_t v) { return (float)v; }
template <typename E> __device__ __forceinline__ E from_f32(float v);
template <> __device__ __forceinline__ float from_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16_t from_f32<bf16_t>(float v) { return (bf16_t)v; }

template <typename E> struct Vec8;  // 8 consecutive elements
template <> struct Vec8<bf16_t> {
  bf16x8_t v;
  __device__ __forceinline__ void load(const bf16_t *p) { v = *reinterpret_cast<const bf16x8_t *>(p); }
  __device__ __forceinline__ void store(bf16_t *p) const { *reinterpret_cast<bf16x8_t *>(p) = v; }
  __device__ __forceinline__ float get(int i) const { return (float)v[i]; }
  __device__ __forceinline__ void set(int i, float f) { v[i] = (bf16_t)f; }
};
template <> struct Vec8<float> {
  float4 a, b;
  __device__ __forceinline__ void load(const float *p) {
    a = *reinterpret_cast<const float4 *>(p);
    b = *reinterpret_cast<const float4 *>(p + 4);
  }
  __device__ __forceinline__ void store(float *p) const {
    *reinterpret_cast<float4 *>(p) = a;
    *reinterpret_cast<float4 *>(p + 4) = b;
  }
  __device__ __forceinline__ float get(int i) const {
    const float *q = i < 4 ? &a.x : &b.x;
    return q[i & 3];
  }
  __device__ __forceinline__ void set(int i, float f) {
    float *q = i < 4 ? &a.x : &b.x;
    q[i & 3] = f;
  }
};

// ---- GEMM engine:  C[M,N] = sum over segments  A_s[M,K_s] * B_s[N,K_s]^T -----------------
// Both operands are K-contiguous ("NT").  K_s % 8 == 0, lda/ldb % 8 == 0, 16-byte aligned
// bases.  C is written in the storage dtype or as float32.
struct GemmSeg {
  const void *A;
  const void *B;
  int64_t lda, ldb;
  int K;
};
struct GemmProblem {
  GemmSeg seg[3];
  int nseg;
  int M, N;
  void *C;
  int64_t ldc;
  int c_f32;  // 1: C is float32 regardless of the storage dtype
  int by_rows;   // fp32 storage, one segment: waves per row, each sum over 64 lanes (the router's logits)
};
// Enqueue up to GEMM_MAX_PROBLEMS independent problems in one launch (N and the output type may
// differ per problem; M too when the launch qualifies for the large-tile bf16 kernel, i.e. every
// M > 128, some N > 128 and every operand below 4 GiB - otherwise differing M is an error).
// scratch (may be empty): room for the fp32 partial tiles of a launch whose last round of tiles is
// cut along K; more than GEMM_SCRATCH_FLOATS is never used, with less fewer cuts are made.
constexpr int GEMM_MAX_PROBLEMS = 8;
constexpr size_t GEMM_SCRATCH_FLOATS = (size_t)256 * 256 * 256;   // one 256 x 256 tile per CU
struct GemmScratch {
  float *part;
  size_t floats;
};
// only >= 0: that problem alone is computed, with the kernel and the cuts it has in the launch of all, so
// that its sums are taken in the same order.
hipError_t launch_gemm(int dtype, const GemmProblem *probs, int nprob, hipStream_t st,
                       const GemmScratch &scratch = GemmScratch{nullptr, 0}, int only = -1);
// the row kernel with the rank-r term of the down projection added, for one or two tokens
struct FewRank;
// the few-rows kernel over K slices of the down projection, and the rank term's sums in further workgroups
bool gemm_few_rank_ok(int dtype, int M, int N, int K);
hipError_t launch_gemm_few_rank(const GemmProblem *probs, int nprob, const FewRank &rank, hipStream_t st);
bool gemm_rows_rank_ok(int dtype, int M, int K);
hipError_t launch_gemm_rows_rank(const GemmProblem &p, const FewRank &rank, hipStream_t st);
// whether products of M rows over a contraction of K go to the row kernel (no need to cut K)
bool gemm_rows_ok(int dtype, int M, int K);
// whether problems of different M may share one launch_gemm call
bool gemm_mixed_rows_ok(int dtype, const GemmProblem *probs, int nprob);

// Measurement hook (csrc/prof.hip): HIP-event timing of launches by kind between prof_begin and
// prof_end (events are recorded on the launch stream).  Not thread-safe; off by default.
// Work is floating-point operations for PROF_GEMM (the DMA-ring bf16 MFMA kernels that carry the
// frozen projections) and algorithmic bytes for the bandwidth-bound kinds.
enum ProfKind {
  PROF_GEMM = 0,      // frozen-projection GEMM launches
  PROF_FUSED_FWD,     // per-pair SwiGLU stage, forward
  PROF_FUSED_BWD,     // per-pair SwiGLU stage, backward
  PROF_COMBINE,       // weighted / unweighted sums of a token's pair rows
  PROF_GRAD_SUMS,     // grouped outer-product sums (LoRA and router gradients)
  PROF_ROUTING,       // softmax / top-k, grouping, auxiliary loss, router backward
  PROF_OTHER,         // re-layouts, gathers, small reductions
  PROF_KINDS
};
bool prof_on();
int prof_begin(int max_launches);
int prof_mark_begin(int kind, hipStream_t st);            // returns a slot (or -1 when off / full)
void prof_mark_end(int slot, hipStream_t st, double work);
int prof_end();
int prof_kind(int kind, double *ms_total, int *launches, double *work_total);

// ---- few tokens (csrc/fused_few.hip; the rank term also in csrc/gemm.hip's row kernel) -----------
constexpr int FEW_MAX_TOKENS = 128, FEW_MAX_PAIRS = 256, FEW_MAX_EXPERTS = 32;
bool few_pairs_ok(int T, int N, int k, int r);
int few_column_blocks(int f);
size_t few_part_floats(int f, int kT, int r);   // floats of Q_part
// Routing from the logits Z, grouping, Eq. 8-9, the per-pair stage, A_down projections (Q_part
// [column block][grouped row][r]) and the weighted combination; bf16 storage.
struct FewStage {
  const float *Z;
  const int32_t *token_model;
  int T, N, Nl, k, r, f;
  float s, coeff;
  int mode;
  const bf16_t *G, *U, *B_gate, *B_up, *A_down;
  const float *Pg_all, *Pu_all;
  bf16_t *a_comb;
  float *Q_part;
  float *probs, *w_out, *w_ws, *loss, *F, *P;
  int32_t *idx_out, *idx_ws, *counts, *counts_out, *offs, *row_of_pair, *pair_of_row, *tok_offs, *model_tokens;
};
hipError_t launch_few_stage(const FewStage &a, hipStream_t st);
// The rank-r term of the down projection from the stage's partial sums; writes Q_all like the other stages.
struct FewRank {
  const float *Q_part, *w;
  const int32_t *idx, *row_of_pair;
  const bf16_t *B_down;
  float *Q_all, *sums;   // sums [T][FEW_RANK_SUMS]: s w_j Q_j, few rows' down product only
  int T, N, k, r, nblk;
  float s;
};
constexpr int FEW_RANK_SUMS = 64;
hipError_t launch_few_finish(const FewRank &a, const float *part, int S, int d, void *y, hipStream_t st);
// sq[j r + q] = s w_j Q[row of slot j of token t][q] for all threads of the workgroup (k r <= 64); red and sq are in LDS
__device__ __forceinline__ void few_rank_sums(const FewRank &a, int t, bool keep, int nthreads, float *red, float *sq) {
  const int V = a.k * a.r, G = nthreads / V, tid = threadIdx.x;
  const int v = tid % V, g = tid / V, j = v / a.r, q = v % a.r;
  const int row = a.row_of_pair[t * a.k + j];
  if (g < G) {
    const float *src = a.Q_part + (int64_t)row * a.r + q;
    const int64_t step = (int64_t)a.T * a.k * a.r;
    float s = 0.f;
    constexpr int INFLIGHT = 8;
    for (int b = g; b < a.nblk; b += INFLIGHT * G) {
      float x[INFLIGHT];
#pragma unroll
      for (int u = 0; u < INFLIGHT; u++) x[u] = src[(b + u * G < a.nblk ? b + u * G : b) * step];
#pragma unroll
      for (int u = 0; u < INFLIGHT; u++)
        if (b + u * G < a.nblk) s += x[u];
    }
    red[tid] = s;
  }
  __syncthreads();
  if (tid < V) {
    float s = 0.f;
    for (int gg = 0; gg < G; gg++) s += red[gg * V + tid];
    const int e = a.idx[t * a.k + j];
    if (keep) a.Q_all[(int64_t)row * a.N * a.r + e * a.r + q] = s;
    sq[tid] = a.s * a.w[t * a.k + j] * s;
  }
  __syncthreads();
}

// ---- routing -----------------------------------------------------------------------------
// N experts in all; with several adapters (token_model != NULL) token t is routed among the Nl
// experts [token_model[t] * Nl, ... + Nl) of its adapter: probs is 0 elsewhere, idx_out is the
// index inside the adapter, idx_ws the index among all N.
// Routing from logits Z[t, n] (row pitch ldz) that a GEMM launch produced, plus weight re-layout jobs.
struct RelayoutJob;
hipError_t launch_route_logits_relayout(int dtype, const float *Z, int ldz, int T, int N, int k, float *probs,
                                        int32_t *idx_out, float *w_out, int32_t *idx_ws,
                                        float *w_ws, int Nl, const int32_t *token_model,
                                        const RelayoutJob *jobs, int njobs, hipStream_t st);
// Routing from logits Z [T, N], grouping as in launch_group_pairs_aux below (and of the tokens by expert pair with
// pg_tok != NULL) and weight re-layout jobs, in one launch up to ROUTE_INLINE_TOKENS tokens, in two above.
constexpr int ROUTE_MAX_K = 4, ROUTE_GROUP_MAX_PAIRS = 8192, ROUTE_GROUP_MAX_EXPERTS = 16, ROUTE_INLINE_TOKENS = 1024;
struct RouteGroup {
  const float *Z;
  const int32_t *token_model;
  int T, N, Nl, k, mode;
  float coeff;
  float *probs, *w_out, *w_ws, *loss, *F, *P;
  int32_t *idx_out, *idx_ws, *counts, *counts_out, *offs, *row_of_pair, *pair_of_row, *tok_offs,
      *model_tokens, *pg_tok, *pg_tiles, *pg_ntiles;
};
bool route_group_ok(int T, int N, int k);
hipError_t launch_route_group(int dtype, const RouteGroup &a, const RelayoutJob *jobs, int njobs, hipStream_t st);
// Stable grouping of the k*T pairs by expert: counts[N], first_counts[N] (slot-0 histogram), offs[N+1],
// row_of_pair[kT], pair_of_row[kT], and launch_aux_loss (without dprobs); tok_offs gets {0, T}.
hipError_t launch_group_pairs_aux(const int32_t *idx, int T, int N, int k, int32_t *counts,
                                  int32_t *counts_out, int32_t *first_counts, int32_t *offs,
                                  int32_t *row_of_pair, int32_t *pair_of_row, int32_t *tok_offs,
                                  const float *probs, float coeff, int mode, float *loss, float *F,
                                  float *P, int Nl, const int32_t *token_model, int32_t *model_tokens,
                                  hipStream_t st);
// The same over many workgroups, for long token batches (identical row maps; the probability
// sums of Eq. 9 are added in a different, equally fixed order).  scratch:
// group_pairs_scratch_bytes(T, k) bytes.
size_t group_pairs_scratch_bytes(int T, int k);
hipError_t launch_group_pairs_aux_multi(const int32_t *idx, int T, int N, int k, int32_t *counts,
                                        int32_t *counts_out, int32_t *first_counts, int32_t *offs,
                                        int32_t *row_of_pair, int32_t *pair_of_row,
                                        int32_t *tok_offs, const float *probs, float coeff, int mode,
                                        float *loss, float *F, float *P, int Nl,
                                        const int32_t *token_model, int32_t *model_tokens,
                                        void *scratch, hipStream_t st);
// loss[N / Nl], one per adapter (statistics over the adapter's own tokens); model_tokens (may be
// NULL) receives the token count of every adapter.
hipError_t launch_aux_loss(const float *probs, const int32_t *idx, int T, int N, int k,
                           float coeff, int mode, float *loss, float *F, float *P,
                           float *dprobs, int Nl, const int32_t *token_model,
                           int32_t *model_tokens, hipStream_t st);

// ---- element-wise / rank-r pieces -------------------------------------------------------
struct PairCtx {  // device pointers describing the grouped pairs
  const int32_t *offs;         // [N+1]
  const int32_t *pair_of_row;  // [kT]
  const int32_t *row_of_pair;  // [kT]
  const float *w;              // [T,k] routing weights
  const int32_t *idx;          // [T,k]
  int T, N, k, r;
};

// a_grp[row,:] = SiLU(G[t] + s B_gate[e] Pg[t,e]) * (U[t] + s B_up[e] Pu[t,e]),  rows grouped
// (fp32 storage, as the next one)
hipError_t launch_swiglu_fwd(const PairCtx &pc, int f, float s, const void *G,
                             const void *U, const float *Pg_all, const float *Pu_all,
                             const void *B_gate, const void *B_up, void *a_grp,
                             hipStream_t st);
// backward of the above; also the per-(row, column tile) partial sums of <H[t], a_row>
hipError_t launch_swiglu_bwd(const PairCtx &pc, int f, float s, const void *G,
                             const void *U, const float *Pg_all, const float *Pu_all,
                             const void *B_gate, const void *B_up, const void *H,
                             const float *VB_all, const void *A_down, void *dg_grp,
                             void *du_grp, float *dw_part, int n_col_tiles, hipStream_t st);
int swiglu_col_tiles(int f);

// Per-expert column factors of the weight-decomposed variant (magnitude / row norm), float32
// [N, f] each, and (backward only) per-tile partial sums for the magnitude gradients,
// [row tiles][f] each with row tiles = kT / 32 + N.
struct DoraArgs {
  const float *cg, *cu;
  float *dm_part_g, *dm_part_u;
};
// bf16 MFMA fusion of the above with the A_down projection of the row's expert: writes a_grp,
// Q_all[row, e(row)*r + q] and the non-zero blocks of Qw[t, e*r + q] = w * Q (bf16, pitch ldqw;
// the caller zero-fills Qw first).  Q_part is scratch of fused_splits(f, kT) * kT * r floats.
hipError_t launch_swiglu_fwd_mfma(const PairCtx &pc, int f, float s, const void *G, const void *U,
                                  const float *Pg_all, const float *Pu_all, const void *B_gate,
                                  const void *B_up, const void *A_down, void *a_grp,
                                  float *Q_part, float *Q_all, void *Qw, int ldqw,
                                  hipStream_t st, int rows_mode = 0, const DoraArgs *dora = nullptr,
                                  bool reduce_parts = true);   // false: the caller sums Q_part itself
// rows_mode of the fused stages (for the paper's own schedules, Figure 3): bit 0 = G and U hold
// one row per grouped pair row instead of one per token; bit 1 = H likewise; bit 2 = the
// block-sparse operand has one row per grouped pair row (unweighted) instead of one per token.
constexpr int ROWS_GU = 1, ROWS_H = 2, ROWS_SPARSE = 4;

// bf16 MFMA backward of the same stage: dg_grp, du_grp, dw_part[row][split]
// (split count = fused_splits(f, kT)), and per split the rank-r partial products of dg with B_gate and of du
// with B_up, [2][split][kT][r] at rank_part.  AdT = A_down re-laid [N, f, r]; BgT / BuT = B banks re-laid
// [N, r, f].  a_grp != NULL (r <= 16, not weight-decomposed): the pairs' activations as well.
hipError_t launch_swiglu_bwd_mfma(const PairCtx &pc, int f, float s, const void *G, const void *U,
                                  const void *H, const float *Pg_all, const float *Pu_all,
                                  const float *VB_all, const void *B_gate, const void *B_up,
                                  const void *AdT, const void *BgT, const void *BuT, void *dg_grp,
                                  void *du_grp, float *dw_part, float *rank_part, void *a_grp, hipStream_t st,
                                  int rows_mode = 0, const DoraArgs *dora = nullptr);
// Pair-grouped token tiles (csrc/fused_pg.hip) for top-2 routing, N <= PG_MAX_EXPERTS, 128 < T <=
// PG_MAX_TOKENS, r <= 16: tokens are grouped by their unordered expert pair, a workgroup handles
// 32 tokens of one pair (forward: one wavefront computes both experts of its columns; backward: one
// set of wavefronts per expert), G / U (/ H) are fetched from HBM once per token and the sums over
// a token's two pairs are written per token (no combine pass).
// Tables: tok_of_pos [T], tile_info [fused_pg_max_tiles(T, N)][4], ntiles [1] (device int32).
// Forward: a_comb[t] = w_t0 a_t0 + w_t1 a_t1, a_grp only when write_a, Q_all / Qw as above;
// Q_part: fused_pg_splits(f, T, N) * kT * r floats.
constexpr int PG_MAX_EXPERTS = 16;
constexpr int PG_TILE_ROWS = 32;
constexpr int PG_MAX_TOKENS = 1 << 16;
bool fused_pg_ok(const PairCtx &pc, int f);
bool fused_pg_bwd_ok(const PairCtx &pc, int f, int Nl);   // Nl: experts per adapter
int fused_pg_max_tiles(int T, int N);
int fused_pg_splits(int f, int T, int N);
hipError_t launch_group_token_pairs(const PairCtx &pc, int32_t *tok_of_pos, int32_t *tile_info,
                                    int32_t *ntiles, hipStream_t st);
hipError_t launch_swiglu_fwd_pg(const PairCtx &pc, int f, float s, const int32_t *tok_of_pos,
                                const int32_t *tile_info, const int32_t *ntiles, const void *G,
                                const void *U, const float *Pg_all, const float *Pu_all,
                                const void *B_gate, const void *B_up, const void *A_down,
                                void *a_comb, float *Q_part, float *Q_all, void *Qw,
                                int ldqw, hipStream_t st);
// backward on the same tiles: the per-token sums dgsum, dusum of the pairs' dg, du; dw_part [pair row][splits], the
// rank-r partial products [2][splits][kT][r] (splits = fused_pg_bwd_splits(f)); the gradients of B_gate, B_up and
// A_down.  slots: fused_pg_bwd_floats floats of scratch.
int fused_pg_bwd_splits(int f);
size_t fused_pg_bwd_floats(int f, int T, int N, int r);
hipError_t launch_swiglu_bwd_pg(const PairCtx &pc, int f, float s, const int32_t *tok_of_pos,
                                const int32_t *tile_info, const int32_t *ntiles, const void *G,
                                const void *U, const void *H, const float *Pg_all,
                                const float *Pu_all, const float *VB_all, const void *B_gate,
                                const void *B_up, const void *AdT, const void *BgT, const void *BuT,
                                void *dgsum, void *dusum, float *dw_part, float *rank_part, float *slots,
                                float *dB_gate, float *dB_up, float *dA_down, hipStream_t st);
// dense[row, e(row)*r + q] = sum over splits of part[split][row][q] (fixed order); the value (times the
// routing weight if weighted) also goes as bf16 into the block-sparse operand sparse[t(row) or row, e*r + q]
hipError_t launch_reduce_rank_parts(const PairCtx &pc, const float *part, int nsplit, float *dense, void *sparse,
                                    int ld_sparse, int weighted, int by_row, hipStream_t st);
int fused_row_tiles(int kT, int N);   // grid.x of the fused stages
int fused_splits(int f, int kT);   // at most FUSED_MAX_SPLITS
constexpr int FUSED_MAX_SPLITS = 32;

// out[t,:] = sum_j (weighted ? w[t,j] : 1) * in_grp[row_of_pair[t,j], :]
// launch_pair_combine (bf16, weighted) and the one-bank weighted per-token launch_reduce_rank_parts
// as one launch (few tokens; k * r <= 256)
hipError_t launch_pair_combine_reduce(const PairCtx &pc, int width, const void *in_grp, void *out,
                                      const float *part, int nsplit, float *dense, void *sparse,
                                      int ld_sparse, hipStream_t st);
hipError_t launch_pair_combine(int dtype, const PairCtx &pc, int width, const void *in_grp,
                               void *out, int weighted, hipStream_t st);
// dst[row, :] = src[token of grouped row, :]   (width a multiple of 8)
hipError_t launch_gather_rows(int dtype, const PairCtx &pc, int width, const void *src, void *dst,
                              hipStream_t st);
// io[t, c] += s * sum_q P[t, q] * Wt[c, q]   (io [T,C] storage dtype, P [T,r] f32, Wt [C,r])
hipError_t launch_lowrank_add(int dtype, void *io, const float *P, const void *Wt, int T, int C,
                              int r, float s, hipStream_t st);

// out[i] = sum_{s<S} part[s][i], i < n, fixed order (closing step of a split-K GEMM)
hipError_t launch_splitk_reduce(int dtype, const float *part, int S, int64_t n, void *out,
                                hipStream_t st);

// Weight re-layouts (tiny index permutations), batched into one launch:
//   dst[dst0 + i0*d0 + i1*d1 + i2*d2] = scale * src[i0*s0 + i1*s1 + i2*s2]   (0 where i2 >= valid2)
// or, with batched_transpose set,  dst[dst0 + b*d0 + q*d1 + p] = scale * src[b*s0 + p*n2 + q]  for
// b < n0, p < n1, q < n2 (0 where p >= valid2), tiled through LDS.
struct RelayoutJob {
  const void *src;
  void *dst;
  int64_t s0, s1, s2, dst0, d0, d1, d2;
  int n0, n1, n2, valid2;
  float scale;
  int batched_transpose;
  size_t zero_bytes;   // non-zero: the job is a plain zero fill of that many bytes at dst
};
constexpr int RELAYOUT_MAX_JOBS = 8;
hipError_t launch_relayout(int dtype, const RelayoutJob *jobs, int njobs, hipStream_t st);
// bytes (rounded up to a multiple of 16) of zeros at dst
RelayoutJob job_zero_fill(void *dst, size_t bytes);
// bank [N, rows, r] -> out[i, col0 + e*r + q] = scale * bank[e, i, q]   (out pitch ldo)
RelayoutJob job_bank_cat(const void *bank, int N, int rows, int r, float scale, void *out,
                         int ldo, int col0);
// bank [N, rows, r] -> out[e*r + q, i]                                   (out is [N*r, rows])
RelayoutJob job_bank_T(const void *bank, int N, int rows, int r, void *out);
// A bank with another number of rank entries: [N, r_src, width] -> [N, r_dst, width] when
// rank_major, else [N, width, r_src] -> [N, width, r_dst]; the first min(r_src, r_dst) entries are
// copied, the rest (if any) are zeros.  Pads a bank to a whole multiple of 8 rank entries, or cuts
// a padded gradient back.
RelayoutJob job_rank_resize(const void *src, void *dst, int N, int r_src, int r_dst, int width,
                            bool rank_major);
// A [N, r, cols] -> out[c, col0 + e*r + q] = scale * A[e, q, c]
RelayoutJob job_A_cat(const void *A, int N, int r, int cols, float scale, void *out, int ldo,
                      int col0);
// W_router [N, d] -> out[c, col0 + n] = W_router[n, c] for n < N, 0 for N <= n < ncols
RelayoutJob job_router_T(const void *W_router, int N, int d, void *out, int ldo, int col0,
                         int ncols);
hipError_t launch_transpose(int dtype, const void *in, void *out, int rows, int cols,
                            hipStream_t st);

// ---- gradients --------------------------------------------------------------------------
// out[g][q][c] (layout_qc = 1) or out[g][c][q] (0) = scale * sum over rows of group g of
//   small[row, q] * wide[(pair_of_row ? pair_of_row[row] / k : row), c];   groups from offs[0..G].
// fp32 storage; rows is the number of rows of all groups together.  Up to GO_MAX_JOBS sums of any
// shapes in one launch; partials holds the sum of their group_outer_partial_floats.
struct GoJob {
  const int32_t *offs, *pair_of_row;
  const float *small, *wide;
  float *out;
  int G, r, C, k, rows, layout_qc;
  float scale;
};
constexpr int GO_MAX_JOBS = 7;
hipError_t launch_group_outer(const GoJob *jobs, int njobs, float *partials, size_t partial_floats,
                              hipStream_t st);
size_t group_outer_partial_floats(int G, int r, int C, int rows);

// bf16 MFMA version: smallT is the transposed bf16 factor [r][ldT] (ldT % 8 == 0, readable up to
// the next multiple of 16 rows past the last group), wide is bf16 with C % 8 == 0.  Up to
// GOM_MAX_JOBS sums of any shapes go into one launch and one reduction launch; `alike` tells how many
// of them have this job's shape; partials must hold the sum of their
// group_outer_mfma_partial_floats.
struct GomJob {
  const void *smallT;
  const void *wide;
  float *out;
  const int32_t *offs, *pair_of_row;
  int G, r, C, k, rows, ldT, alike, layout_qc;
  float scale;
};
constexpr int GOM_MAX_JOBS = 8;
hipError_t launch_group_outer_mfma(const GomJob *jobs, int njobs, float *partials, size_t partial_floats,
                                   hipStream_t st);
size_t group_outer_mfma_partial_floats(int G, int r, int C, int rows, int alike);
// a per-row rank-r factor: (w_row or 1) * src[(by_token ? t(row) : row), e(row)*r + q], as bf16 at
// outT[q, row] (pitch ldT) or in fp32 storage at outT[row, q]
struct GatherJob {
  const float *src;
  void *outT;
  int by_token, weighted;
};
constexpr int GATHER_MAX_JOBS = 6;
hipError_t launch_f32_to_bf16T(const float *src, int rows, int r, void *outT, int ldT,
                               hipStream_t st);

struct AuxUpstream {   // upstream gradient of every adapter's auxiliary loss
  float v[64];
};
// ---- row-wise steps behind a fused stage, one launch (csrc/tail.hip) ----------------------------------
// Parts that are not wanted are left zero.
struct TailArgs {
  PairCtx pc;
  // router gradient (probs != NULL): dw -> dz, also into columns col0 .. of the K-extension operand S
  const float *probs, *dw_part, *VB_all, *Q_all, *F;
  int n_col_tiles;
  float s, aux_coeff;
  AuxUpstream d_aux;
  float *dw_ws, *dz;
  void *S;
  int ld_s, col0, ncols, Nl;
  const int32_t *token_model, *model_tokens;
  bf16_t *dzT;             // bf16 [N][ldTz] copy or NULL
  int ldTz, s_by_first_pair;   // S has one row per grouped pair row
  // bf16 storage (part != NULL): two banks of rank-r partial products -> S and their transposed factors
  const float *part;
  int64_t bank_stride;
  int nsplit, ldT;
  bf16_t *redT[2];
  // row factors
  GatherJob gather[GATHER_MAX_JOBS];
  int ngather;
  // fp32 storage: block-sparse operand from dense rank-r rows, up to two banks side by side
  const float *scatter_src[2];
  void *scatter_dst;
  int nscatter, ld_scatter, scatter_weighted;
  // sums over a token's pair rows
  const void *comb_in[2];
  void *comb_out[2];
  int ncombine, width, comb_weighted;
};
struct TailBlocks {   // workgroups of each part (of one bank, job, token)
  int router, reduce, gather, scatter, combine, total;
};
hipError_t launch_tail(int dtype, const TailArgs &a, hipStream_t st);

// ---- weight-decomposed experts (csrc/dora.hip); bf16 storage only --------------------------------
hipError_t launch_row_sqnorm(const void *W_gate, const void *W_up, const void *W_down, int f, int d,
                             float *out, hipStream_t st);   // out [2 f + d]
size_t gram_part_floats(int N, int r);   // floats of one bank's Gram slice sums
hipError_t launch_gram(const void *A_gate, const void *A_up, const void *A_down, int N, int r, int f,
                       int d, float *part, hipStream_t st);   // part: 3 * gram_part_floats
// c = m / n, ninv = 1 / n with n the row norms of W + s B_e A_e (from w2, WA = W A_cat^T, AA) for the
// projections gate, up, down
struct DoraScale {
  const void *B_bank;
  const float *WA, *m;
  float *c, *ninv;
};
hipError_t launch_dora_scale(const DoraScale *proj, int shared, int N, int f, int d, int r, float s,
                             const float *AA, const float *w2, hipStream_t st);
hipError_t launch_scale_bank(void *bank, const float *c, int N, int r, int d, hipStream_t st);
hipError_t launch_gather_rows_scaled(const PairCtx &pc, int width, const void *src, const float *c,
                                     void *dst, hipStream_t st);
hipError_t launch_pair_combine_scaled(const PairCtx &pc, int width, const void *in_grp,
                                      const float *c, void *out, hipStream_t st);
size_t dm_down_part_floats(int N, int d);
hipError_t launch_dm_down(const PairCtx &pc, int d, const void *dy, const void *v, const float *ninv,
                          float *part, float *dm, int shared, hipStream_t st);
hipError_t launch_dm_tiles_reduce(const int32_t *offs, int N, int f, const float *part_g,
                                  const float *part_u, const float *ninv_g, const float *ninv_u,
                                  float *dm_g, float *dm_u, int shared, hipStream_t st);

}  // namespace mixlora
