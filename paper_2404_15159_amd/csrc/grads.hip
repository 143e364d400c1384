// Gradient kernels: sums of outer products over the rows of each expert group (the LoRA A/B
// gradients and the router weight gradient), and the router's backward (top-k renormalised
// softmax of Eq. 7 / Algorithm 1 plus the auxiliary term of Eq. 8-9).
//
// Each LoRA gradient has the form  out[g] = scale * sum_{rows of group g} small[row] (x) wide[row']
// with `small` an r-vector per grouped row and `wide` a d- or d_ff-wide row (grouped, or the
// token's row).  The sum over rows is split into fixed slices whose partial results are added
// in a fixed order by a second kernel: no floating-point atomics, bit-reproducible.
#include "common.h"

#include <type_traits>

namespace mixlora {

constexpr int GO_COLS = 512;   // 256 threads x 2 adjacent columns
constexpr int GO_STAGE = 64;   // rows staged per pass

// fp32 storage: all sums of a pass in one launch (each alone is little more than a launch's latency).
struct GoBatch {
  GoJob job[GO_MAX_JOBS];
  float *partial[GO_MAX_JOBS];
  int nsplit[GO_MAX_JOBS], y0[GO_MAX_JOBS];   // y0: first blockIdx.y of the job
  int njobs;
};

// partial[split][g][q][c], q < r.  RQ = rank chunk held in registers.  blockIdx.y = y0 of the job +
// split * G + group.
template <int RQ>
__global__ __launch_bounds__(256) void group_outer_kernel(GoBatch batch) {
  __shared__ float sm[GO_STAGE][RQ];
  __shared__ int src_s[GO_STAGE];
  int ji = 0;
  while (ji + 1 < batch.njobs && batch.y0[ji + 1] <= (int)blockIdx.y) ji++;
  const GoJob &J = batch.job[ji];
  const int G = J.G, r = J.r, C = J.C, nsplit = batch.nsplit[ji];
  if ((int)blockIdx.x * GO_COLS >= C) return;
  const int g = (blockIdx.y - batch.y0[ji]) % G, sp = (blockIdx.y - batch.y0[ji]) / G;
  const int lo = J.offs[g], hi = J.offs[g + 1];
  const int len = (hi - lo + nsplit - 1) / nsplit;
  const int r_lo = lo + sp * len;
  const int r_hi = r_lo + len < hi ? r_lo + len : hi;
  const int c = blockIdx.x * GO_COLS + threadIdx.x * 2;
  const bool active = c < C;
  for (int q0 = 0; q0 < r; q0 += RQ) {
    float acc[RQ][2];
#pragma unroll
    for (int q = 0; q < RQ; q++) acc[q][0] = acc[q][1] = 0.f;
    for (int rb = r_lo; rb < r_hi; rb += GO_STAGE) {
      const int n = r_hi - rb < GO_STAGE ? r_hi - rb : GO_STAGE;
      __syncthreads();
      for (int i = threadIdx.x; i < GO_STAGE * RQ; i += 256) {
        const int rr = i / RQ, q = i % RQ;
        sm[rr][q] = (rr < n && q0 + q < r) ? J.small[(int64_t)(rb + rr) * r + q0 + q] : 0.f;
      }
      if (threadIdx.x < GO_STAGE && threadIdx.x < n)
        src_s[threadIdx.x] = J.pair_of_row ? J.pair_of_row[rb + threadIdx.x] / J.k : rb + threadIdx.x;
      __syncthreads();
      if (active) {
#pragma unroll 4
        for (int rr = 0; rr < n; rr++) {
          const float2 v = *reinterpret_cast<const float2 *>(J.wide + (int64_t)src_s[rr] * C + c);
#pragma unroll
          for (int q = 0; q < RQ; q++) {
            const float sv = sm[rr][q];
            acc[q][0] = fmaf(sv, v.x, acc[q][0]);
            acc[q][1] = fmaf(sv, v.y, acc[q][1]);
          }
        }
      }
    }
    if (active) {
#pragma unroll
      for (int q = 0; q < RQ; q++) {
        if (q0 + q < r) {
          float *o = batch.partial[ji] + (((int64_t)sp * G + g) * r + q0 + q) * C + c;
          *reinterpret_cast<float2 *>(o) = make_float2(acc[q][0], acc[q][1]);
        }
      }
    }
  }
}

// out = scale * sum of the job's partials in split order, written as [g][q][c] or [g][c][q]
__global__ __launch_bounds__(256) void group_outer_sum_kernel(GoBatch batch) {
  const GoJob &J = batch.job[blockIdx.y];
  const int64_t n = (int64_t)J.G * J.r * J.C;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float *__restrict__ partial = batch.partial[blockIdx.y] + i;
  float acc = 0.f;
#pragma unroll 4
  for (int sp = 0; sp < batch.nsplit[blockIdx.y]; sp++) acc += partial[sp * n];
  acc *= J.scale;
  if (J.layout_qc) {
    J.out[i] = acc;
  } else {
    const int c = (int)(i % J.C), q = (int)((i / J.C) % J.r), g = (int)(i / ((int64_t)J.C * J.r));
    J.out[((int64_t)g * J.C + c) * J.r + q] = acc;
  }
}

// Row slices of a job: enough workgroups for the chip, at least 16 rows of an average group each
// (a slice of two rows costs more in partial sums than it saves).
static int go_splits(int G, int C, int rows) {
  const int col_tiles = (C + GO_COLS - 1) / GO_COLS;
  int s = 1024 / (col_tiles * G);
  if (s > rows / (16 * G)) s = rows / (16 * G);
  if (s > 32) s = 32;
  return s < 1 ? 1 : s;
}

size_t group_outer_partial_floats(int G, int r, int C, int rows) {
  return (size_t)go_splits(G, C, rows) * G * r * C;
}

hipError_t launch_group_outer(const GoJob *jobs, int njobs, float *partials, size_t partial_floats,
                              hipStream_t st) {
  if (njobs < 1 || njobs > GO_MAX_JOBS) return hipErrorInvalidValue;
  GoBatch b{};
  b.njobs = njobs;
  size_t used = 0;
  int y = 0, x = 0, rmax = 0;
  int64_t n = 0;
  for (int i = 0; i < njobs; i++) {
    const GoJob &J = jobs[i];
    b.job[i] = J;
    b.nsplit[i] = go_splits(J.G, J.C, J.rows);
    b.partial[i] = partials + used;
    used += (size_t)b.nsplit[i] * J.G * J.r * J.C;
    b.y0[i] = y;
    y += J.G * b.nsplit[i];
    const int ct = (J.C + GO_COLS - 1) / GO_COLS;
    x = ct > x ? ct : x;
    rmax = J.r > rmax ? J.r : rmax;
    const int64_t m = (int64_t)J.G * J.r * J.C;
    n = m > n ? m : n;
  }
  if (used > partial_floats) return hipErrorInvalidValue;
  if (rmax > 8) hipLaunchKernelGGL(group_outer_kernel<16>, dim3(x, y), dim3(256), 0, st, b);
  else hipLaunchKernelGGL(group_outer_kernel<8>, dim3(x, y), dim3(256), 0, st, b);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(group_outer_sum_kernel, dim3((unsigned)((n + 255) / 256), njobs), dim3(256), 0, st, b);
  return hipGetLastError();
}

// ---- bf16 MFMA version of the grouped outer-product sums ----------------------------------------
// out[g][q][c] partial = sum over a slice of group g's rows of smallT[q][row] * wide[src(row)][c].
// The contraction index is the row: first MFMA operand = wide (index = column, 8 rows per
// lane, read as 2-byte-pair loads whose even/odd halves feed two column-interleaved MFMA
// blocks), second operand = smallT (index = q, 8 consecutive rows = one 16-byte load from the
// transposed bf16 copy).  Rows outside the group are masked in the small operand.
constexpr int GOM_CB = 8;     // column blocks per wave: a lane reads 8 adjacent columns (16 bytes)

// A wave covers 256 columns: lane (l31, hi) reads, for each of its 8 rows, the 16-byte run of
// columns c0 + 8*l31 .. +7; element b of the run feeds MFMA block b, whose operand index i = l31
// therefore stands for column c0 + 8*i + b.  In the result, lane (q, hi) register 4*gg + m of
// block b is column c0 + 8*(8*gg + 4*hi + m) + b: for fixed (gg, m) the 8 blocks give 8
// consecutive columns, stored as two float4.
// All sums of a pass share one launch (blockIdx.x = first block of the job + (split * G + group) *
// column groups + column group): the wide ones come first, and the short ones, which alone left most
// of the chip waiting, fill in behind them.  Against one launch per shape and a reduction each: 187 ->
// 147 us at the 7B shape, 55 -> 30 at 300 tokens.
struct GomBatch {
  GomJob job[GOM_MAX_JOBS];
  float *partial[GOM_MAX_JOBS];
  int nsplit[GOM_MAX_JOBS], x0[GOM_MAX_JOBS];
  int njobs;
};

template <int NQ>
__global__ __launch_bounds__(256, NQ == 1 ? 2 : 1) void group_outer_mfma_kernel(GomBatch batch) {
  int ji = 0;
  while (ji + 1 < batch.njobs && batch.x0[ji + 1] <= (int)blockIdx.x) ji++;
  const GomJob &J = batch.job[ji];
  const int G = J.G, r = J.r, C = J.C, ldT = J.ldT, nsplit = batch.nsplit[ji], nrows = J.rows, k = J.k;
  const int cgs = (C + 1023) >> 10, at = blockIdx.x - batch.x0[ji];
  const int cg = at % cgs, g = at / cgs % G, sp = at / cgs / G;
  const bf16_t *__restrict__ smallT = reinterpret_cast<const bf16_t *>(J.smallT);
  const bf16_t *__restrict__ wide = reinterpret_cast<const bf16_t *>(J.wide);
  const int32_t *__restrict__ pair_of_row = J.pair_of_row;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l31 = lane & 31, hi = lane >> 5;
  const int lo = J.offs[g], hi_ = J.offs[g + 1];
  const int base = lo & ~15;
  const int nsteps = hi_ > lo ? (hi_ - base + 15) >> 4 : 0;
  const int per = (nsteps + nsplit - 1) / nsplit;
  const int st_lo = sp * per;
  const int st_hi = st_lo + per < nsteps ? st_lo + per : nsteps;
  const int c0 = (cg * 4 + wave) * (32 * GOM_CB);
  if (c0 >= C) return;   // whole wave out of range (no barriers in this kernel)
  int ccol = c0 + 8 * l31;
  if (ccol >= C) ccol = C - 8;
  f32x16_t acc[GOM_CB][NQ];
#pragma unroll
  for (int b = 0; b < GOM_CB; b++)
#pragma unroll
    for (int j = 0; j < NQ; j++)
#pragma unroll
      for (int i = 0; i < 16; i++) acc[b][j][i] = 0.f;

  auto walk = [&](auto gather) {
  for (int st = st_lo; st < st_hi; st++) {
    const int rbase = base + st * 16 + hi * 8;
    bf16x8_t bq[NQ];
#pragma unroll
    for (int j = 0; j < NQ; j++) {
      const int q = j * 32 + l31;
      bq[j] = *reinterpret_cast<const bf16x8_t *>(smallT + (int64_t)(q < r ? q : 0) * ldT + rbase);
    }
    // rows read in place are read exactly once per step: a streaming (non-temporal) load keeps them from
    // displacing the gathered rows and partial results other kernels reuse (the sums over the d_ff-wide
    // operands measured 28 % faster); gathered token rows are read by k groups and stay cached
    bf16x8_t wrow[8];
#pragma unroll
    for (int p = 0; p < 8; p++) {
      const int row = rbase + p < nrows ? rbase + p : nrows - 1;
      if constexpr (decltype(gather)::value)
        wrow[p] = *reinterpret_cast<const bf16x8_t *>(wide + (int64_t)(pair_of_row[row] / k) * C + ccol);
      else
        wrow[p] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8_t *>(wide + (int64_t)row * C + ccol));
    }
    __builtin_amdgcn_sched_barrier(0);   // every load of the step is on its way before the masks
#pragma unroll
    for (int j = 0; j < NQ; j++) {
      const bool qv = j * 32 + l31 < r;
#pragma unroll
      for (int p = 0; p < 8; p++) {
        const int row = rbase + p;
        bq[j][p] = (qv & (row >= lo) & (row < hi_)) ? bq[j][p] : (bf16_t)0.f;
      }
    }
#pragma unroll
    for (int b = 0; b < GOM_CB; b++) {
      bf16x8_t fa;
#pragma unroll
      for (int p = 0; p < 8; p++) fa[p] = wrow[p][b];
#pragma unroll
      for (int j = 0; j < NQ; j++)
        acc[b][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, bq[j], acc[b][j], 0, 0, 0);
    }
  }
  };
  if (pair_of_row) walk(std::true_type{});   // (decided outside the loop)
  else walk(std::false_type{});
  const float scale = J.scale;
#pragma unroll
  for (int j = 0; j < NQ; j++) {
    const int q = j * 32 + l31;
    if (q < r) {
      if (nsplit == 1) {
        // rows not split: scale and write the result itself, [g][q][c] or [g][c][q]
        float *out = J.out;
        const bool qc = J.layout_qc != 0;
#pragma unroll
        for (int gg = 0; gg < 4; gg++)
#pragma unroll
          for (int m = 0; m < 4; m++) {
            const int c = c0 + 8 * (8 * gg + 4 * hi + m);
            if (c + 7 < C) {
              if (qc) {
                float *o = out + ((int64_t)g * r + q) * C + c;
                *reinterpret_cast<float4 *>(o) =
                    make_float4(scale * acc[0][j][gg * 4 + m], scale * acc[1][j][gg * 4 + m],
                                scale * acc[2][j][gg * 4 + m], scale * acc[3][j][gg * 4 + m]);
                *reinterpret_cast<float4 *>(o + 4) =
                    make_float4(scale * acc[4][j][gg * 4 + m], scale * acc[5][j][gg * 4 + m],
                                scale * acc[6][j][gg * 4 + m], scale * acc[7][j][gg * 4 + m]);
              } else {
                float *o = out + ((int64_t)g * C + c) * r + q;
#pragma unroll
                for (int b = 0; b < GOM_CB; b++) o[(int64_t)b * r] = scale * acc[b][j][gg * 4 + m];
              }
            }
          }
        continue;
      }
      float *o = batch.partial[ji] + (((int64_t)sp * G + g) * r + q) * C;
#pragma unroll
      for (int gg = 0; gg < 4; gg++)
#pragma unroll
        for (int m = 0; m < 4; m++) {
          const int c = c0 + 8 * (8 * gg + 4 * hi + m);
          if (c + 7 < C) {
            *reinterpret_cast<float4 *>(o + c) = make_float4(acc[0][j][gg * 4 + m], acc[1][j][gg * 4 + m],
                                                             acc[2][j][gg * 4 + m], acc[3][j][gg * 4 + m]);
            *reinterpret_cast<float4 *>(o + c + 4) = make_float4(acc[4][j][gg * 4 + m], acc[5][j][gg * 4 + m],
                                                                 acc[6][j][gg * 4 + m], acc[7][j][gg * 4 + m]);
          }
        }
    }
  }
}

// out = scale * sum of a split job's partials in split order; blockIdx.y picks the job.  One element per
// thread, reads along the columns, eight slices in flight (four rank entries per thread, for 16-byte
// stores of the [g][c][q] form, left too few threads: 42 against 11 us at the 7B shape).
__global__ __launch_bounds__(256) void group_outer_reduce_kernel(GomBatch batch) {
  const GomJob &J = batch.job[blockIdx.y];
  const int nsplit = batch.nsplit[blockIdx.y], r = J.r, C = J.C;
  const int64_t n = (int64_t)J.G * r * C;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (nsplit == 1 || i >= n) return;
  const float *src = batch.partial[blockIdx.y] + i;
  float acc = 0.f;
  for (int s0 = 0; s0 < nsplit; s0 += 8) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; u++) v[u] = src[(int64_t)(s0 + u < nsplit ? s0 + u : s0) * n];
#pragma unroll
    for (int u = 0; u < 8; u++)
      if (s0 + u < nsplit) acc += v[u];
  }
  acc *= J.scale;
  if (J.layout_qc) {
    J.out[i] = acc;
  } else {
    const int c = (int)(i % C), q = (int)(i / C % r), g = (int)(i / ((int64_t)C * r));
    J.out[((int64_t)g * C + c) * r + q] = acc;
  }
}

// Row slices of a job, `alike` jobs of its shape being in the launch: enough workgroups that they cover
// the chip twice (256 CUs x 2 workgroups of 4 waves), and at least 64 rows of an average group each -
// a slice's partial sums cost a trip through memory and back.
static int gom_splits(int G, int C, int rows, int alike) {
  const int cgs = (C + 1023) / 1024;
  int s = 512 / (cgs * G * alike);
  if (s > 8 && G > 1) s = 8;
  // one group beside others (the router's sum): 12 slices are as good as 32 there (1 % on the step), but a
  // few workgroups that walk more than 512 rows each outlast the rest of the launch
  const int beside = rows > 6144 ? rows / 512 : 12, alone = 32;
  if (G == 1 && s > (alike == 1 ? beside : alone)) s = alike == 1 ? beside : alone;
  if (s > 64) s = 64;
  if (s > rows / (64 * G)) s = rows / (64 * G);
  return s < 1 ? 1 : s;
}

size_t group_outer_mfma_partial_floats(int G, int r, int C, int rows, int alike) {
  const int s = gom_splits(G, C, rows, alike);
  return s > 1 ? (size_t)s * G * r * C : 0;
}

hipError_t launch_group_outer_mfma(const GomJob *jobs, int njobs, float *partials, size_t partial_floats,
                                   hipStream_t st) {
  if (njobs < 1 || njobs > GOM_MAX_JOBS) return hipErrorInvalidValue;
  // Jobs that cover the chip twice by themselves keep a launch of their own (L3-8B shape, 672
  // workgroups of d_ff-wide sums: 0.6 % on the step against one launch for all).
  int lead = 0;
  for (int64_t wgs = 0; lead < njobs && jobs[lead].C == jobs[0].C && jobs[lead].G == jobs[0].G; lead++) {
    wgs += (jobs[lead].C + 1023) / 1024 * jobs[lead].G * gom_splits(jobs[lead].G, jobs[lead].C, jobs[lead].rows, jobs[lead].alike);
    if (lead + 1 == jobs[0].alike && lead + 1 < njobs && wgs > 512) {
      size_t used = 0;
      for (int i = 0; i <= lead; i++)
        used += group_outer_mfma_partial_floats(jobs[i].G, jobs[i].r, jobs[i].C, jobs[i].rows, jobs[i].alike);
      if (used > partial_floats) return hipErrorInvalidValue;
      const hipError_t e = launch_group_outer_mfma(jobs, lead + 1, partials, used, st);
      if (e != hipSuccess) return e;
      return launch_group_outer_mfma(jobs + lead + 1, njobs - lead - 1, partials + used, partial_floats - used, st);
    }
  }
  GomBatch b{};
  b.njobs = njobs;
  size_t used = 0;
  int x = 0, rmax = 0;
  int64_t n = 0;   // reduction threads of the largest split job
  for (int i = 0; i < njobs; i++) {
    const GomJob &J = jobs[i];
    b.job[i] = J;
    b.nsplit[i] = gom_splits(J.G, J.C, J.rows, J.alike);
    b.partial[i] = partials + used;
    used += group_outer_mfma_partial_floats(J.G, J.r, J.C, J.rows, J.alike);
    b.x0[i] = x;
    x += (J.C + 1023) / 1024 * J.G * b.nsplit[i];
    rmax = J.r > rmax ? J.r : rmax;
    const int64_t m = b.nsplit[i] > 1 ? (int64_t)J.G * J.r * J.C : 0;
    n = m > n ? m : n;
  }
  if (used > partial_floats) return hipErrorInvalidValue;
  if (rmax <= 32) hipLaunchKernelGGL(group_outer_mfma_kernel<1>, dim3(x), dim3(256), 0, st, b);
  else hipLaunchKernelGGL(group_outer_mfma_kernel<2>, dim3(x), dim3(256), 0, st, b);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || n == 0) return e;   // unsplit rows: the kernel wrote the results
  hipLaunchKernelGGL(group_outer_reduce_kernel, dim3((unsigned)((n + 255) / 256), njobs), dim3(256), 0, st, b);
  return hipGetLastError();
}

// outT[q][row] (bf16) = src[row][q] (fp32, [rows, r])
__global__ void f32_to_bf16T_kernel(const float *__restrict__ src, int rows, int r,
                                    bf16_t *__restrict__ outT, int ldT) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)rows * r) return;
  const int q = (int)(i / rows), row = (int)(i % rows);
  outT[(int64_t)q * ldT + row] = (bf16_t)src[(int64_t)row * r + q];
}

hipError_t launch_f32_to_bf16T(const float *src, int rows, int r, void *outT, int ldT,
                               hipStream_t st) {
  const int64_t n = (int64_t)rows * r;
  hipLaunchKernelGGL(f32_to_bf16T_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, src,
                     rows, r, (bf16_t *)outT, ldT);
  return hipGetLastError();
}

}  // namespace mixlora
