// Few tokens (decode-shaped calls): everything between the gate/up product and the down product in one
// launch, and the down product's rank-r term added where its K slices are.
//
// What bounds these calls beside the weight stream is the number of launches: each costs 4-5 us however
// little it does, and routing, grouping, the per-pair stage, the weighted combination and the sum of the
// rank-r partial products were four of them.  With at most 256 pairs the routing is cheaper to repeat in
// every workgroup than to hand over: a lane routes one token, a ballot per bit of the expert's index
// groups the pairs.  A workgroup owns 64 columns of d_ff for ALL pairs, so the weighted sum of a
// token's activations (Algorithm 1 line 15) stays inside it; its eight waves take the
// experts in turn, 32 rows at a time, with the MFMA roles of csrc/fused.hip, each finding its experts' rows
// from the pairs' expert numbers by itself (no barrier but the one behind the routing).
// 7B block: one token, four launches 22.2 us -> one of 6.8 (69.8 -> 58.4 us per pass); 64 tokens 25.9 -> 9.6 and
// 4.8 for the closing sum (82.8 -> 71.5 per pass).  Asking for the LoRA weights in front of the routing costs
// 2 us: they are waited for at the routing's barrier, and experts without a token are read too.  Summing the
// rank-r partial products (one per column block) in the closing launch costs 4 us more than in workgroups
// of the down product's launch, where it is hidden.
#include "fused_common.h"
#include "route_lane.h"

namespace mixlora {

namespace {
constexpr int FEW_WAVES = 8;
}  // namespace

bool few_pairs_ok(int T, int N, int k, int r) {
  return T <= FEW_MAX_TOKENS && T * k <= FEW_MAX_PAIRS && N <= FEW_MAX_EXPERTS && k <= ROUTE_MAX_K && r <= 16;
}
int few_column_blocks(int f) { return (f + FT_SB - 1) / FT_SB; }
size_t few_part_floats(int f, int kT, int r) { return (size_t)few_column_blocks(f) * kT * r; }

template <int NMAX>
__global__ __launch_bounds__(FEW_WAVES * 64) void few_stage_kernel(FewStage a, int nblk) {
  extern __shared__ __align__(16) unsigned char dyn[];
  constexpr int CH = FEW_MAX_PAIRS / 64;
  __shared__ int eid[FEW_MAX_PAIRS], rowof[FEW_MAX_PAIRS], tokof[FEW_MAX_PAIRS];   // tokof: token of a grouped row
  __shared__ float wgt[FEW_MAX_PAIRS];
  const int T = a.T, N = a.N, k = a.k, r = a.r, R = N * r, f = a.f, kT = k * T;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool meta = (int)blockIdx.x == nblk;   // the last workgroup writes the routing tables and Eq. 8-9
  float *ps = reinterpret_cast<float *>(dyn);  // there: probabilities [T][N]

  // ---- routing: thread t, token t
  if (tid < T) {
    float z[NMAX], p[NMAX], ws[ROUTE_MAX_K];
    int es[ROUTE_MAX_K];
#pragma unroll
    for (int n = 0; n < NMAX; n++) z[n] = a.Z[(int64_t)tid * N + (n < N ? n : 0)];
    const int lo = a.token_model ? a.token_model[tid] * a.Nl : 0;
    if (meta) route_lane<NMAX, true>(z, lo, a.Nl, k, p, es, ws);
    else route_lane<NMAX, false>(z, lo, a.Nl, k, p, es, ws);
#pragma unroll
    for (int j = 0; j < ROUTE_MAX_K; j++)
      if (j < k) {
        eid[tid * k + j] = es[j];
        wgt[tid * k + j] = ws[j];
      }
    if (meta) {
#pragma unroll
      for (int n = 0; n < NMAX; n++)
        if (n < N) ps[tid * N + n] = p[n];
    }
  }
  int tok[CH];   // token of pair 64 c + lane
#pragma unroll
  for (int c = 0; c < CH; c++) tok[c] = (64 * c + lane) / k;
  __syncthreads();
  // ---- grouping, by every wave for the experts it takes: rows of one expert are consecutive, experts in
  // ascending order, rows in ascending pair order
  int ep[CH];
#pragma unroll
  for (int c = 0; c < CH; c++) ep[c] = 64 * c + lane < kT ? eid[64 * c + lane] : FEW_MAX_EXPERTS;
  const unsigned long long lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  auto count_rows = [&](int ex, int &row0, int &n) {
    row0 = n = 0;
#pragma unroll
    for (int c = 0; c < CH; c++) {
      row0 += __popcll(__ballot(ep[c] < ex));
      n += __popcll(__ballot(ep[c] == ex));
    }
  };
  auto place_rows = [&](int ex, int row) {
#pragma unroll
    for (int c = 0; c < CH; c++) {
      const unsigned long long m = __ballot(ep[c] == ex);
      if (ep[c] == ex) {
        const int at = row + __popcll(m & lt);
        rowof[64 * c + lane] = at;
        tokof[at] = tok[c];
      }
      row += __popcll(m);
    }
  };
  // eight waves and fewer experts: several waves per expert, its tiles in turn
  const int span = N > 4 ? 8 : N > 2 ? 4 : N > 1 ? 2 : 1, turns = FEW_WAVES / span;
  const int turn = wave / span;

  if (meta) {
    for (int ex = wave; ex < N; ex += FEW_WAVES) {
      int row0, n, fc = 0, Tm = T;
      count_rows(ex, row0, n);
      place_rows(ex, row0);
      for (int t = lane; t < T; t += 64) fc += eid[t * k] == ex;
      if (a.token_model) {
        Tm = 0;
        for (int t = lane; t < T; t += 64) Tm += a.token_model[t] == ex / a.Nl;
      }
      float sum = 0.f;
      for (int t = lane; t < T; t += 64) sum += ps[t * N + ex];
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        fc += __shfl_xor(fc, o, 64);
        if (a.token_model) Tm += __shfl_xor(Tm, o, 64);
        sum += __shfl_xor(sum, o, 64);
      }
      if (lane == 0) {
        a.counts[ex] = a.counts_out[ex] = n;
        a.offs[ex] = row0;
        if (ex % a.Nl == 0) a.model_tokens[ex / a.Nl] = Tm;
        const bool top1 = a.mode == MIXLORA_AUX_TOP1;
        const float denom = top1 ? (float)Tm : (float)Tm * (float)k;
        const float P = Tm > 0 ? sum / (float)Tm : 0.f, F = Tm > 0 ? (float)(top1 ? fc : n) / denom : 0.f;
        a.P[ex] = P;
        a.F[ex] = F;
        ps[T * N + ex] = F * P;
      }
    }
    __syncthreads();
    if (tid < kT) {
      const int lo = a.token_model ? a.token_model[tid / k] * a.Nl : 0, row = rowof[tid];
      a.idx_out[tid] = eid[tid] - lo;
      a.idx_ws[tid] = eid[tid];
      a.w_out[tid] = a.w_ws[tid] = wgt[tid];
      a.row_of_pair[tid] = row;
      a.pair_of_row[row] = tid;
    }
    for (int i = tid; i < T * N; i += FEW_WAVES * 64) a.probs[i] = ps[i];
    if (tid < N / a.Nl) {
      float acc = 0.f;
      for (int n = 0; n < a.Nl; n++) acc += ps[T * N + tid * a.Nl + n];
      a.loss[tid] = a.coeff * (float)a.Nl * acc;
    }
    if (tid == 0) {
      a.offs[N] = kT;
      a.tok_offs[0] = 0;
      a.tok_offs[1] = T;
    }
    return;
  }

  // ---- per-pair stage: activations of all pairs in this workgroup's columns, [kT][FT_PITCH]
  bf16_t *at = reinterpret_cast<bf16_t *>(dyn);
  bf16_t *tu = at + kT * FT_PITCH + wave * FT_TILE;   // this wave's tile of the up projection's deltas
  const int l31 = lane & 31, hi = lane >> 5, rr = lane >> 3, cc = lane & 7;
  const int c0 = blockIdx.x * FT_SB, q0 = hi * 8;
  const bool v = q0 < r;
  const int col = c0 + 8 * cc, colr = col < f ? col : f - 8;
  for (int ex = wave % span; ex < N; ex += span) {
    int first, n;
    count_rows(ex, first, n);
    if (n <= turn * FT_ROWS) continue;
    bf16x8_t wg[2], wu[2], wf[4];
#pragma unroll
    for (int b = 0; b < 2; b++) {
      int cw = c0 + 32 * b + l31;
      cw = cw < f ? cw : f - 1;
      const int64_t o = ((int64_t)ex * f + cw) * r + (v ? q0 : 0);
      wg[b] = ld8(a.B_gate + o);
      wu[b] = ld8(a.B_up + o);
    }
#pragma unroll
    for (int s4 = 0; s4 < 4; s4++) {
      int cw = c0 + 16 * s4 + 8 * hi;
      cw = cw < f ? cw : f - 8;
      wf[s4] = ld8(a.A_down + ((int64_t)ex * r + (l31 < r ? l31 : 0)) * f + cw);
    }
    place_rows(ex, first);
    __builtin_amdgcn_wave_barrier();
    for (int t0 = turn * FT_ROWS; t0 < n; t0 += turns * FT_ROWS) {
      const int row0 = first + t0, rows = n - t0 < FT_ROWS ? n - t0 : FT_ROWS;
      const int64_t tm = tokof[row0 + (l31 < rows ? l31 : 0)];
      const int64_t po = tm * R + ex * r + (v ? q0 : 0);
      const bf16x8_t pg = cvt8(a.Pg_all + po, v, a.s), pu = cvt8(a.Pu_all + po, v, a.s);
      bf16x8_t gv[4], uv[4];
#pragma unroll
      for (int p = 0; p < 4; p++) {
        const int rl = 8 * p + rr;
        const int64_t o = (int64_t)tokof[row0 + (rl < rows ? rl : 0)] * f + colr;
        gv[p] = ld8(a.G + o);
        uv[p] = ld8(a.U + o);
      }
#pragma unroll
      for (int b = 0; b < 2; b++) {
        f32x16_t dg, du;
#pragma unroll
        for (int i = 0; i < 16; i++) dg[i] = du[i] = 0.f;
        dg = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wg[b], pg, dg, 0, 0, 0);
        du = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wu[b], pu, du, 0, 0, 0);
        if (l31 < rows) tile_put(at + row0 * FT_PITCH, l31, hi, 32 * b, dg);   // rows past it are another tile's
        tile_put(tu, l31, hi, 32 * b, du);
      }
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int p = 0; p < 4; p++) {
        const int rl = 8 * p + rr;
        if (rl < rows) {
          bf16_t *tp = at + (row0 + rl) * FT_PITCH + 8 * cc;
          const bf16x8_t dgl = ld8(tp), dul = ld8(tu + rl * FT_PITCH + 8 * cc);
          bf16x8_t av;
#pragma unroll
          for (int m = 0; m < 8; m++) {
            const float gg = (float)gv[p][m] + (float)dgl[m];
            const float uu = (float)uv[p][m] + (float)dul[m];
            av[m] = (bf16_t)(gg * fsigmoid(gg) * uu);   // columns past f: finite, meet zeroed weights
          }
          *reinterpret_cast<bf16x8_t *>(tp) = av;
        }
      }
      __builtin_amdgcn_wave_barrier();
      // partial sums over these columns of a[row, c] A_down[ex, q, c]
      f32x16_t accq;
#pragma unroll
      for (int i = 0; i < 16; i++) accq[i] = 0.f;
#pragma unroll
      for (int s4 = 0; s4 < 4; s4++) {
        const bf16x8_t af = ld8(at + (row0 + (l31 < rows ? l31 : 0)) * FT_PITCH + 16 * s4 + 8 * hi);
        bf16x8_t w = wf[s4];
        if (c0 + 16 * s4 + 8 * hi >= f) w = zero8();
        accq = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af, w, accq, 0, 0, 0);
      }
      if (l31 < r) {
        float *q = a.Q_part + ((int64_t)blockIdx.x * kT + row0 + 4 * hi) * r + l31;
#pragma unroll
        for (int i = 0; i < 16; i++) {
          const int rl = 8 * (i >> 2) + (i & 3);
          if (rl + 4 * hi < rows) q[rl * r] = accq[i];
        }
      }
    }
  }
  __syncthreads();
  // ---- weighted combination, slots in order (the activations themselves are not stored: a backward pass makes
  // them again; storing them costs a forward of 64 tokens of the 7B block 1 us of 72)
  for (int i = tid; i < T * 8; i += FEW_WAVES * 64) {
    const int t = i >> 3, c = c0 + 8 * (i & 7);
    if (c >= f) continue;
    float s[8];
#pragma unroll
    for (int m = 0; m < 8; m++) s[m] = 0.f;
    for (int j = 0; j < k; j++) {
      const bf16x8_t v = ld8(at + rowof[t * k + j] * FT_PITCH + 8 * (i & 7));
      const float w = wgt[t * k + j];
#pragma unroll
      for (int m = 0; m < 8; m++) s[m] = fmaf(w, (float)v[m], s[m]);
    }
    bf16x8_t o;
#pragma unroll
    for (int m = 0; m < 8; m++) o[m] = (bf16_t)s[m];
    *reinterpret_cast<bf16x8_t *>(a.a_comb + (int64_t)t * f + c) = o;
  }
}

hipError_t launch_few_stage(const FewStage &a, hipStream_t st) {
  if (!few_pairs_ok(a.T, a.N, a.k, a.r)) return hipErrorInvalidValue;
  const int nblk = few_column_blocks(a.f), kT = a.k * a.T;
  size_t smem = (size_t)(kT * FT_PITCH + FEW_WAVES * FT_TILE) * sizeof(bf16_t);
  const size_t meta = ((size_t)a.T * a.N + a.N) * sizeof(float);
  smem = smem > meta ? smem : meta;
  auto kern = a.N <= 8 ? few_stage_kernel<8> : a.N <= 16 ? few_stage_kernel<16> : few_stage_kernel<32>;
  static bool attr_set[3] = {false, false, false};
  const int inst = a.N <= 8 ? 0 : a.N <= 16 ? 1 : 2;
  if (!attr_set[inst]) {
    constexpr int most = (FEW_MAX_PAIRS * FT_PITCH + FEW_WAVES * FT_TILE) * (int)sizeof(bf16_t);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, most);
    if (e != hipSuccess) return e;
    attr_set[inst] = true;
  }
  hipLaunchKernelGGL(kern, dim3(nblk + 1), dim3(FEW_WAVES * 64), smem, st, a, nblk);
  return hipGetLastError();
}

// y[t, c] = sum over the K slices of the down product, in slice order, + sum_j w_j s (Q_j B_down[e_j]^T)[c]
// with s w_j Q_j from the down product's launch.  A workgroup: one token, 512 columns.
__global__ __launch_bounds__(256) void few_finish_kernel(FewRank a, const float *__restrict__ part, int S, int d,
                                                         bf16_t *__restrict__ y) {
  const int t = blockIdx.y, c = blockIdx.x * 512 + threadIdx.x * 2;
  const bool in = c < d;   // d is even
  const int cr = in ? c : 0;
  const int r = a.r;
  bf16x8_t b[ROUTE_MAX_K][2][2];   // [slot][column][half of the rank]
#pragma unroll
  for (int j = 0; j < ROUTE_MAX_K; j++)
    if (j < a.k) {
      const bf16_t *src = a.B_down + ((int64_t)a.idx[t * a.k + j] * d + cr) * r;
#pragma unroll
      for (int i = 0; i < 2; i++)
#pragma unroll
        for (int h = 0; h < 2; h++) b[j][i][h] = ld8(src + i * r + (h * 8 < r ? h * 8 : 0));
    }
  float acc[2] = {0.f, 0.f};
  const int64_t step = (int64_t)a.T * d;
  for (int sl = 0; sl < S; sl++) {
    const float2 v = *reinterpret_cast<const float2 *>(part + sl * step + (int64_t)t * d + cr);
    acc[0] += v.x;
    acc[1] += v.y;
  }
  const float *sq = a.sums + t * FEW_RANK_SUMS;
#pragma unroll
  for (int j = 0; j < ROUTE_MAX_K; j++)
    if (j < a.k)
#pragma unroll
      for (int h = 0; h < 2; h++)
        if (h * 8 < r)
#pragma unroll
          for (int m = 0; m < 8; m++) {
            const float q = sq[j * r + h * 8 + m];
            acc[0] = fmaf(q, (float)b[j][0][h][m], acc[0]);
            acc[1] = fmaf(q, (float)b[j][1][h][m], acc[1]);
          }
  if (in) {
    typedef bf16_t bf16x2_t __attribute__((ext_vector_type(2)));
    bf16x2_t o;
    o[0] = (bf16_t)acc[0];
    o[1] = (bf16_t)acc[1];
    *reinterpret_cast<bf16x2_t *>(y + (int64_t)t * d + c) = o;
  }
}

hipError_t launch_few_finish(const FewRank &a, const float *part, int S, int d, void *y, hipStream_t st) {
  hipLaunchKernelGGL(few_finish_kernel, dim3((d + 511) / 512, a.T), dim3(256), 0, st, a, part, S, d, (bf16_t *)y);
  return hipGetLastError();
}

}  // namespace mixlora
