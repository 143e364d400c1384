// The row-wise steps behind a fused stage, as block ranges of one launch: they depend on that stage (fp32
// storage: on the small product behind it) and not on each other, and at 300 tokens each is little more
// than a launch's own 4-5 us.  Backward: router gradient, sums over column splits of the rank-r partial
// products (bf16), per-row rank-r factors of the gradient sums, per-token sums of dg and du, block-sparse
// low-rank operand (fp32); forward, fp32 storage: the last one and the weighted combine.  Four or five launches
// in one: a step at the 7B block with 300 tokens 383.7 -> 372.8 us, with 1999 of rank 32 1367 -> 1349, the small
// fp32 configuration 101.9 -> 92.7; 2000 tokens, top-3, 1024 x 2752: 343.6 -> 326.2.
#include "row_bodies.h"

namespace mixlora {

// ---- router backward -------------------------------------------------------------------------
// One wavefront per token.  dw_j = <dy_t, o_pair> is assembled from the column-tile partials of
// <H[t], a_row> plus the low-rank part  s <B_down[e]^T dy_t, A_down[e] a_row>  (lanes split the
// terms, a butterfly adds them).  Then, with w_j = p_j / sum_kept p (Norm of Algorithm 1):
// dp_j = (dw_j - sum_i w_i dw_i) / sum_kept p on the kept experts, plus the auxiliary term
// d_aux * a * N * F_e / T  on every expert (Eq. 8-9; F is piecewise constant; evaluated as its
// deviation from 1/N, see below), and
// dz = p * (dp - <p, dp>) through the softmax of Eq. 7 (lane e holds expert e).  With several
// adapters p is zero outside the token's adapter, so dz is too; T and the upstream gradient of
// the auxiliary loss are those of the token's adapter.
__device__ __forceinline__ float rb_wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

template <typename E>
__device__ __forceinline__ void router_bwd_body(const TailArgs &a, int block) {
  const int lane = threadIdx.x & 63;
  const PairCtx &pc = a.pc;
  const int t = block * 4 + (threadIdx.x >> 6);
  if (t >= pc.T) return;   // whole wave leaves together
  const int N = pc.N, k = pc.k, r = pc.r, R = N * r;
  float my_dw = 0.f, my_w = 0.f, my_p = 0.f;   // lane j < k: slot j of the token
  int my_e = -1;
  for (int j = 0; j < k; j++) {
    const int p = t * k + j;
    const int row = pc.row_of_pair[p];
    const int e = pc.idx[p];
    float part = 0.f;
    for (int ct = lane; ct < a.n_col_tiles; ct += 64) part += a.dw_part[(int64_t)row * a.n_col_tiles + ct];
    float lr = 0.f;
    for (int q = lane; q < r; q += 64)
      lr = fmaf(a.VB_all[(int64_t)t * R + e * r + q], a.Q_all[(int64_t)row * R + e * r + q], lr);
    const float dwj = rb_wave_sum(part + a.s * lr);
    if (lane == j) {
      my_dw = dwj;
      my_e = e;
      my_w = pc.w[p];
      my_p = a.probs[(int64_t)t * N + e];
      a.dw_ws[p] = dwj;
    }
  }
  const float wdw = rb_wave_sum(my_w * my_dw);
  const float ssum = rb_wave_sum(my_p);
  // auxiliary term of the token's adapter: statistics over that adapter's own tokens
  const int m = __builtin_amdgcn_readfirstlane(a.token_model ? a.token_model[t] : 0);   // wave-uniform
  const float auxg = a.d_aux.v[m] * a.aux_coeff * (float)a.Nl / (float)a.model_tokens[m];
  // The softmax Jacobian ignores a constant added to dp, so F_e - 1/a.Nl stands in for F_e: with
  // nearly balanced loads (what the loss drives towards) p * (F_e - <p, F>) would otherwise be a
  // difference of nearly equal numbers.  F_e * (k * tokens) is an integer in both modes of Eq. 9
  // (k times the first-slot count, or the kept count), recovered exactly by rounding, so the
  // deviation (num_e * a.Nl - k * tokens) / (k * tokens * a.Nl) has an exact numerator.
  float dp = 0.f;
  if (lane < N) {
    const float kt = (float)k * (float)a.model_tokens[m];
    const int64_t num = (int64_t)rintf(a.F[lane] * kt);
    const int64_t dev = num * a.Nl - (int64_t)k * a.model_tokens[m];
    dp = auxg * ((float)dev / (kt * (float)a.Nl));
  }
  for (int j = 0; j < k; j++) {
    const int ej = __shfl(my_e, j, 64);
    const float dwj = __shfl(my_dw, j, 64);
    if (ej == lane) dp += (dwj - wdw) / ssum;
  }
  const float pe = lane < N ? a.probs[(int64_t)t * N + lane] : 0.f;
  const float dot = rb_wave_sum(pe * dp);
  const float v = pe * (dp - dot);   // 0 on lanes >= N
  if (lane < N) {
    a.dz[(int64_t)t * N + lane] = v;
    // transposed bf16 copy: the row factor of the dW_router outer-product sum
    if (a.dzT) a.dzT[(int64_t)lane * a.ldTz + t] = (bf16_t)v;
  }
  // row of the K-extension operand: the token's, or (operand with one row per grouped pair row)
  // the row of the token's first slot, whose other rows keep zeros in these columns
  const int64_t srow = a.s_by_first_pair ? pc.row_of_pair[t * pc.k] : t;
  for (int e = lane; e < a.ncols; e += 64)
    reinterpret_cast<E *>(a.S)[srow * a.ld_s + a.col0 + e] = from_f32<E>(e < N ? v : 0.f);
}

// Rank-r partial products summed over the column splits, 256 / r rows per block: bf16 into the
// block-sparse operand, and (through LDS) into the transposed row factor of the gradient sums.
__device__ __forceinline__ void reduce_body(const TailArgs &a, int bank, int block, bf16_t *tile) {
  const PairCtx &pc = a.pc;
  const int r = pc.r, nP = pc.T * pc.k, rb = 256 / r, row0 = block * rb, i = threadIdx.x;
  const int rl = i / r, q = i % r, row = row0 + rl;
  if (rl < rb && row < nP) {
    const float *part = a.part + bank * a.bank_stride + (int64_t)row * r + q;
    const int64_t step = (int64_t)nP * r;
    float acc = 0.f;
    int sp = 0;
    for (; sp + 8 <= a.nsplit; sp += 8) {   // eight loads in flight; additions in split order
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; u++) v[u] = part[(sp + u) * step];
#pragma unroll
      for (int u = 0; u < 8; u++) acc += v[u];
    }
    for (; sp < a.nsplit; sp++) acc += part[sp * step];
    const int pair = pc.pair_of_row[row], e = pc.idx[pair];
    reinterpret_cast<bf16_t *>(a.S)[(int64_t)(a.s_by_first_pair ? row : pair / pc.k) * a.ld_s +
                                    bank * pc.N * r + e * r + q] = (bf16_t)acc;
    tile[q * (rb + 1) + rl] = (bf16_t)acc;
  }
  __syncthreads();
  const int qo = i / rb, ro = i % rb;
  if (qo < r && row0 + ro < nP) a.redT[bank][(int64_t)qo * a.ldT + row0 + ro] = tile[qo * (rb + 1) + ro];
}

// out[row, q] = (w_row or 1) * src[(by_token ? t(row) : row), e(row) r + q]; bf16: transposed, out[q][row]
template <typename E>
__device__ __forceinline__ void gather_body(const TailArgs &a, const GatherJob &J, int block, bf16_t *tile) {
  const PairCtx &pc = a.pc;
  const int r = pc.r, nP = pc.T * pc.k, rb = 256 / r, row0 = block * rb, i = threadIdx.x;
  const int rl = i / r, q = i % r, row = row0 + rl;
  if (rl < rb && row < nP) {
    const int p = pc.pair_of_row[row], e = pc.idx[p];
    const int64_t srow = J.by_token ? p / pc.k : row;
    const float v = (J.weighted ? pc.w[p] : 1.f) * J.src[srow * (pc.N * r) + e * r + q];
    if constexpr (sizeof(E) == 2) tile[q * (rb + 1) + rl] = (bf16_t)v;
    else reinterpret_cast<float *>(J.outT)[(int64_t)row * r + q] = v;
  }
  if constexpr (sizeof(E) == 2) {
    __syncthreads();
    const int qo = i / rb, ro = i % rb;
    if (qo < r && row0 + ro < nP)
      reinterpret_cast<bf16_t *>(J.outT)[(int64_t)qo * a.ldT + row0 + ro] = tile[qo * (rb + 1) + ro];
  }
}

// dst[t, bank N r + e r + q] = (w_j or 1) * src_bank[row_j, e r + q] when expert e is slot j of token t, else 0
__device__ __forceinline__ void scatter_body(const TailArgs &a, int bank, int block) {
  const PairCtx &pc = a.pc;
  const int R = pc.N * pc.r;
  const int64_t i = (int64_t)block * 256 + threadIdx.x;
  if (i >= (int64_t)pc.T * R) return;
  const int t = (int)(i / R), er = (int)(i % R), e = er / pc.r;
  float v = 0.f;
  for (int j = 0; j < pc.k; j++) {
    const int p = t * pc.k + j;
    if (pc.idx[p] == e)
      v = (a.scatter_weighted ? pc.w[p] : 1.f) * a.scatter_src[bank][(int64_t)pc.row_of_pair[p] * R + er];
  }
  reinterpret_cast<float *>(a.scatter_dst)[(int64_t)t * a.ld_scatter + bank * R + er] = v;
}

// Workgroups in rows of TAIL_GRID_X: a grid dimension holds less than 2^32 threads, and millions of tokens of a
// narrow block need more workgroups than that in one.
constexpr int TAIL_GRID_X = 1 << 16;

template <typename E>
__global__ __launch_bounds__(256) void tail_kernel(TailArgs a, TailBlocks n) {
  __shared__ bf16_t tile[256 + 64];
  int b = blockIdx.y * TAIL_GRID_X + blockIdx.x;   // all branches are workgroup-uniform
  if (b >= n.total) return;
  if (b < n.router) {
    router_bwd_body<E>(a, b);
    return;
  }
  b -= n.router;
  if constexpr (sizeof(E) == 2) {
    if (b < 2 * n.reduce) {
      reduce_body(a, b >= n.reduce, b >= n.reduce ? b - n.reduce : b, tile);
      return;
    }
    b -= 2 * n.reduce;
  }
  if (b < a.ngather * n.gather) {
    gather_body<E>(a, a.gather[b / n.gather], b % n.gather, tile);
    return;
  }
  b -= a.ngather * n.gather;
  if constexpr (sizeof(E) == 4) {
    if (b < a.nscatter * n.scatter) {
      scatter_body(a, b / n.scatter, b % n.scatter);
      return;
    }
    b -= a.nscatter * n.scatter;
  }
  const int slices = n.combine, per = a.pc.T * slices, which = b / per, x = b - which * per;
  pair_combine_body<E>(a.pc, a.width, reinterpret_cast<const E *>(a.comb_in[which]),
                       reinterpret_cast<E *>(a.comb_out[which]), a.comb_weighted, x / slices, x % slices);
}

hipError_t launch_tail(int dtype, const TailArgs &a, hipStream_t st) {
  const PairCtx &pc = a.pc;
  const int nP = pc.T * pc.k, rb = 256 / pc.r;
  TailBlocks n{};
  n.router = a.probs ? (pc.T + 3) / 4 : 0;
  n.reduce = a.part ? (nP + rb - 1) / rb : 0;
  n.gather = a.ngather ? (nP + rb - 1) / rb : 0;
  n.scatter = a.nscatter ? (int)(((int64_t)pc.T * pc.N * pc.r + 255) / 256) : 0;
  n.combine = a.ncombine ? pair_combine_slices(a.width) : 0;
  if (pc.r > 64 || a.ngather > GATHER_MAX_JOBS || a.nscatter > 2 || a.ncombine > 2 ||
      (dtype == MIXLORA_BF16 ? a.nscatter : n.reduce))
    return hipErrorInvalidValue;
  const int64_t blocks = n.router + 2ll * n.reduce + (int64_t)a.ngather * n.gather + (int64_t)a.nscatter * n.scatter +
                         (int64_t)a.ncombine * n.combine * pc.T;
  static_assert((int64_t)TAIL_GRID_X * 256 < (1ll << 32) && (1ll << 31) / TAIL_GRID_X < 65536, "grid limits");
  if (blocks < 1 || blocks >= (1ll << 31) - TAIL_GRID_X) return hipErrorInvalidValue;
  n.total = (int)blocks;
  const dim3 grid(blocks < TAIL_GRID_X ? (unsigned)blocks : TAIL_GRID_X, (unsigned)((blocks + TAIL_GRID_X - 1) / TAIL_GRID_X));
  if (dtype == MIXLORA_BF16) hipLaunchKernelGGL(tail_kernel<bf16_t>, grid, dim3(256), 0, st, a, n);
  else hipLaunchKernelGGL(tail_kernel<float>, grid, dim3(256), 0, st, a, n);
  return hipGetLastError();
}

}  // namespace mixlora
