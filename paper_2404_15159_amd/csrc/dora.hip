// Pieces of the weight-decomposed expert variant ("MixDoRA" in the paper's experiments, which
// gives no formula; the reading follows the cited weight-decomposition method): every expert
// projection is  diag(m_e / n_e) (W + s B_e A_e),  n_e = row norms of W + s B_e A_e, held constant
// in the backward pass.  The frozen product stays shared; the per-expert factor c_e = m_e / n_e is
// applied to the rows of the routed pairs.  bf16 storage only.
//
// Row norms without forming W + s B_e A_e:
//   n_e[j]^2 = |W[j,:]|^2 + 2 s B_e[j,:] . (W A_e^T)[j,:] + s^2 B_e[j,:] (A_e A_e^T) B_e[j,:]^T
// with W A_e^T from the GEMM engine (rank-r output columns) and the r x r Gram matrices and the
// squared row norms of W from the small kernels below.
#include "common.h"

namespace mixlora {

// ---- w2[j] = sum_i W[j, i]^2, one wavefront per row, lanes in a fixed order ---------------------
// The three frozen matrices in one launch (270 MB at the 7B shape, HBM-bound): w2 holds the rows of
// W_gate, W_up and W_down one after the other.
__global__ __launch_bounds__(256) void row_sqnorm_kernel(const bf16_t *__restrict__ Wg,
                                                         const bf16_t *__restrict__ Wu,
                                                         const bf16_t *__restrict__ Wd, int f, int d,
                                                         float *__restrict__ out) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= 2 * f + d) return;
  const bf16_t *p = row < f       ? Wg + (int64_t)row * d
                    : row < 2 * f ? Wu + (int64_t)(row - f) * d
                                  : Wd + (int64_t)(row - 2 * f) * f;
  const int cols = row < 2 * f ? d : f;
  float acc = 0.f;
#pragma unroll 4
  for (int c = lane * 8; c < cols; c += 64 * 8) {
    const bf16x8_t v = *reinterpret_cast<const bf16x8_t *>(p + c);
#pragma unroll
    for (int i = 0; i < 8; i++) acc = fmaf((float)v[i], (float)v[i], acc);
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if (lane == 0) out[row] = acc;
}

hipError_t launch_row_sqnorm(const void *W_gate, const void *W_up, const void *W_down, int f, int d,
                             float *out, hipStream_t st) {
  hipLaunchKernelGGL(row_sqnorm_kernel, dim3((2 * f + d + 3) / 4), dim3(256), 0, st,
                     (const bf16_t *)W_gate, (const bf16_t *)W_up, (const bf16_t *)W_down, f, d, out);
  return hipGetLastError();
}

// ---- AA[b][e][q][q'] = sum_i A_b[e, q, i] A_b[e, q', i]  (banks A_gate, A_up, A_down) -----------
// MFMA 16x16x32 with both operands straight from memory (the bank is its own transpose's K-major
// form).  The input dimension is cut into GRAM_SLICES slices of eight waves each; slice sums go to
// part[b][slice][e][q][q'] and are added in slice order by the consumer.  All banks in one launch:
// bound by a chain of a few loads per wave (68 -> 8 us against one launch per bank with r^2 scalar
// products from LDS, 7B shape, 8 experts of rank 16).
constexpr int GRAM_SLICES = 4;

template <int NQ>
__global__ __launch_bounds__(512) void gram_kernel(const bf16_t *__restrict__ Ag,
                                                   const bf16_t *__restrict__ Au,
                                                   const bf16_t *__restrict__ Ad, int r, int f, int d,
                                                   int N, float *__restrict__ part) {
  __shared__ float red[8][NQ][64][4];
  const int e = blockIdx.x, sl = blockIdx.y, b = blockIdx.z;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l15 = lane & 15, hi = lane >> 4;
  const int in = b == 2 ? f : d;
  const bf16_t *A = (b == 0 ? Ag : b == 1 ? Au : Ad) + (int64_t)e * r * in;
  float *out = part + (((int64_t)b * GRAM_SLICES + sl) * N + e) * r * r;
  const bf16_t *ar[NQ];
#pragma unroll
  for (int j = 0; j < NQ; j++) ar[j] = A + (int64_t)(j * 16 + l15 < r ? j * 16 + l15 : r - 1) * in;
  f32x4_t acc[NQ][NQ];
#pragma unroll
  for (int i = 0; i < NQ; i++)
#pragma unroll
    for (int j = 0; j < NQ; j++) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  for (int k0 = (sl * 8 + wave) * 32; k0 < in; k0 += GRAM_SLICES * 8 * 32) {
    const int k = k0 + hi * 8;
    bf16x8_t fr[NQ];
#pragma unroll
    for (int j = 0; j < NQ; j++) {
      fr[j] = *reinterpret_cast<const bf16x8_t *>(ar[j] + (k < in ? k : 0));
      if (k >= in) {   // in % 8 == 0
#pragma unroll
        for (int m = 0; m < 8; m++) fr[j][m] = (bf16_t)0.f;
      }
    }
#pragma unroll
    for (int i = 0; i < NQ; i++)
#pragma unroll
      for (int j = 0; j < NQ; j++)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fr[j], fr[i], acc[i][j], 0, 0, 0);
  }
  // acc[i][j][m] of lane (l15, hi): q = 16 i + l15, q' = 16 j + 4 hi + m
#pragma unroll
  for (int i = 0; i < NQ; i++) {
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NQ; j++) *reinterpret_cast<f32x4_t *>(red[wave][j][lane]) = acc[i][j];
    __syncthreads();
    for (int x = threadIdx.x; x < NQ * 256; x += 512) {
      const int j = x >> 8, ln = (x >> 2) & 63, m = x & 3;
      const int q = i * 16 + (ln & 15), q2 = j * 16 + (ln >> 4) * 4 + m;
      float v = red[0][j][ln][m];
#pragma unroll
      for (int w = 1; w < 8; w++) v += red[w][j][ln][m];
      if (q < r && q2 < r) out[q * r + q2] = v;
    }
  }
}

size_t gram_part_floats(int N, int r) { return (size_t)GRAM_SLICES * N * r * r; }

hipError_t launch_gram(const void *A_gate, const void *A_up, const void *A_down, int N, int r, int f,
                       int d, float *part, hipStream_t st) {
  const dim3 grid(N, GRAM_SLICES, 3), block(512);
#define MIXLORA_GRAM(NQ_)                                                                       \
  hipLaunchKernelGGL(gram_kernel<NQ_>, grid, block, 0, st, (const bf16_t *)A_gate,              \
                     (const bf16_t *)A_up, (const bf16_t *)A_down, r, f, d, N, part)
  if (r <= 16) MIXLORA_GRAM(1);
  else if (r <= 32) MIXLORA_GRAM(2);
  else MIXLORA_GRAM(4);
#undef MIXLORA_GRAM
  return hipGetLastError();
}

// ---- c[e, j] = m[e, j] / n_e[j],  ninv[e, j] = 1 / n_e[j] ----------------------------------------
// B banks [N, out, r] bf16; WA [out, N*r] float32; AA: the Gram kernel's slice sums; w2 as above;
// c, ninv [N, out]; m [N, out] or one [out] vector shared by the experts.  The three projections in
// one launch (blockIdx.z); a thread owns one output feature and keeps its r bank entries in registers.
struct DoraScaleJob {
  const bf16_t *B;
  const float *WA, *AA, *w2, *m;
  int out;
  float *c, *ninv;
};
struct DoraScaleBatch {
  DoraScaleJob job[3];
};

template <int RMAX>
__global__ __launch_bounds__(256) void dora_scale_kernel(DoraScaleBatch batch, int shared, int N, int r,
                                                         float s) {
  __shared__ float aa[RMAX * RMAX];
  const DoraScaleJob &J = batch.job[blockIdx.z];
  const int e = blockIdx.y, out = J.out;
  if ((int)blockIdx.x * 256 >= out) return;
  for (int i = threadIdx.x; i < r * r; i += 256) {
    float a = 0.f;
#pragma unroll
    for (int sl = 0; sl < GRAM_SLICES; sl++) a += J.AA[((int64_t)sl * N + e) * r * r + i];
    aa[i] = a;
  }
  __syncthreads();
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j >= out) return;
  const bf16_t *b = J.B + ((int64_t)e * out + j) * r;
  const float *wa = J.WA + (int64_t)j * N * r + e * r;
  float bv[RMAX];
  float cross = 0.f, quad = 0.f;
#pragma unroll
  for (int q0 = 0; q0 < RMAX; q0 += 8) {   // r % 8 == 0
    if (q0 < r) {
      Vec8<bf16_t> v;
      Vec8<float> w;
      v.load(b + q0);
      w.load(wa + q0);
#pragma unroll
      for (int q = 0; q < 8; q++) {
        bv[q0 + q] = v.get(q);
        cross = fmaf(v.get(q), w.get(q), cross);
      }
    } else {
#pragma unroll
      for (int q = 0; q < 8; q++) bv[q0 + q] = 0.f;
    }
  }
#pragma unroll
  for (int q = 0; q < RMAX; q++) {
    if (q < r) {
      float row = 0.f;
#pragma unroll
      for (int q2 = 0; q2 < RMAX; q2++)
        if (q2 < r) row = fmaf(aa[q * r + q2], bv[q2], row);
      quad = fmaf(bv[q], row, quad);
    }
  }
  const float n2 = J.w2[j] + 2.f * s * cross + s * s * quad;
  const float inv = n2 > 0.f ? 1.f / sqrtf(n2) : 0.f;
  J.ninv[(int64_t)e * out + j] = inv;
  J.c[(int64_t)e * out + j] = J.m[(shared ? 0 : (int64_t)e * out) + j] * inv;
}

hipError_t launch_dora_scale(const DoraScale *p, int shared, int N, int f, int d, int r, float s,
                             const float *AA, const float *w2, hipStream_t st) {
  DoraScaleBatch b;
  const int out[3] = {f, f, d}, w2_at[3] = {0, f, 2 * f};
  for (int i = 0; i < 3; i++)
    b.job[i] = DoraScaleJob{(const bf16_t *)p[i].B_bank, p[i].WA, AA + i * gram_part_floats(N, r), w2 + w2_at[i],
                            p[i].m, out[i], p[i].c, p[i].ninv};
  const dim3 grid(((f > d ? f : d) + 255) / 256, N, 3), block(256);
  if (r <= 8) hipLaunchKernelGGL(dora_scale_kernel<8>, grid, block, 0, st, b, shared, N, r, s);
  else if (r <= 16) hipLaunchKernelGGL(dora_scale_kernel<16>, grid, block, 0, st, b, shared, N, r, s);
  else if (r <= 32) hipLaunchKernelGGL(dora_scale_kernel<32>, grid, block, 0, st, b, shared, N, r, s);
  else hipLaunchKernelGGL(dora_scale_kernel<64>, grid, block, 0, st, b, shared, N, r, s);
  return hipGetLastError();
}

// ---- bank[(e*r + q), j] *= c[e, j]   (transposed B_down bank [N*r, d]) ---------------------------
__global__ void scale_bank_kernel(bf16_t *__restrict__ bank, const float *__restrict__ c, int N,
                                  int r, int d) {
  const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 8;
  if (i >= (int64_t)N * r * d) return;
  const int row = (int)(i / d), j = (int)(i % d);
  const int e = row / r;
  bf16x8_t v = *reinterpret_cast<bf16x8_t *>(bank + i);
#pragma unroll
  for (int q = 0; q < 8; q++) v[q] = (bf16_t)((float)v[q] * c[(int64_t)e * d + j + q]);
  *reinterpret_cast<bf16x8_t *>(bank + i) = v;
}

hipError_t launch_scale_bank(void *bank, const float *c, int N, int r, int d, hipStream_t st) {
  const int64_t n = (int64_t)N * r * d / 8;
  hipLaunchKernelGGL(scale_bank_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
                     (bf16_t *)bank, c, N, r, d);
  return hipGetLastError();
}

// ---- dst[row, :] = c[e(row), :] * src[token of row, :] -------------------------------------------
__global__ __launch_bounds__(256) void gather_rows_scaled_kernel(PairCtx pc, int width,
                                                                 const bf16_t *__restrict__ src,
                                                                 const float *__restrict__ c,
                                                                 bf16_t *__restrict__ dst) {
  const int row = blockIdx.x;
  const int col = (blockIdx.y * 256 + threadIdx.x) * 8;
  if (col >= width) return;
  const int pair = pc.pair_of_row[row];
  const int e = pc.idx[pair];
  bf16x8_t v = *reinterpret_cast<const bf16x8_t *>(src + (int64_t)(pair / pc.k) * width + col);
#pragma unroll
  for (int q = 0; q < 8; q++) v[q] = (bf16_t)((float)v[q] * c[(int64_t)e * width + col + q]);
  *reinterpret_cast<bf16x8_t *>(dst + (int64_t)row * width + col) = v;
}

hipError_t launch_gather_rows_scaled(const PairCtx &pc, int width, const void *src, const float *c,
                                     void *dst, hipStream_t st) {
  const dim3 grid(pc.T * pc.k, (width / 8 + 255) / 256), block(256);
  hipLaunchKernelGGL(gather_rows_scaled_kernel, grid, block, 0, st, pc, width, (const bf16_t *)src,
                     c, (bf16_t *)dst);
  return hipGetLastError();
}

// ---- out[t, :] = sum_j w[t, j] * c[e_j, :] * in_grp[row_of_pair[t, j], :]  (slots ascending) -----
__global__ __launch_bounds__(256) void pair_combine_scaled_kernel(PairCtx pc, int width,
                                                                  const bf16_t *__restrict__ in_grp,
                                                                  const float *__restrict__ c,
                                                                  bf16_t *__restrict__ out) {
  const int t = blockIdx.x;
  const int col = (blockIdx.y * 256 + threadIdx.x) * 8;
  if (col >= width) return;
  float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int j = 0; j < pc.k; j++) {
    const int p = t * pc.k + j;
    const float w = pc.w[p];
    const float *ce = c + (int64_t)pc.idx[p] * width + col;
    const bf16x8_t v = *reinterpret_cast<const bf16x8_t *>(in_grp + (int64_t)pc.row_of_pair[p] * width + col);
#pragma unroll
    for (int i = 0; i < 8; i++) acc[i] = fmaf(w * ce[i], (float)v[i], acc[i]);
  }
  bf16x8_t o;
#pragma unroll
  for (int i = 0; i < 8; i++) o[i] = (bf16_t)acc[i];
  *reinterpret_cast<bf16x8_t *>(out + (int64_t)t * width + col) = o;
}

hipError_t launch_pair_combine_scaled(const PairCtx &pc, int width, const void *in_grp,
                                      const float *c, void *out, hipStream_t st) {
  const dim3 grid(pc.T, (width / 8 + 255) / 256), block(256);
  hipLaunchKernelGGL(pair_combine_scaled_kernel, grid, block, 0, st, pc, width,
                     (const bf16_t *)in_grp, c, (bf16_t *)out);
  return hipGetLastError();
}

// ---- magnitude gradient of the down projection ---------------------------------------------------
// dm[e, j] = ninv[e, j] * sum over the rows of expert e of  w_row * dy[token, j] * v[row, j]
// (v = unscaled output of the per-pair down projection).  Rows are cut into DMD_SLICES slices per
// expert; slice sums are written to part[slice][e][j] and added in slice order afterwards.
constexpr int DMD_SLICES = 16;

__global__ __launch_bounds__(256) void dm_down_part_kernel(PairCtx pc, int d,
                                                           const bf16_t *__restrict__ dy,
                                                           const bf16_t *__restrict__ v,
                                                           float *__restrict__ part) {
  const int e = blockIdx.y, sl = blockIdx.z;
  const int col = (blockIdx.x * 256 + threadIdx.x) * 8;
  if (col >= d) return;
  const int lo = pc.offs[e], hi = pc.offs[e + 1];
  const int per = (hi - lo + DMD_SLICES - 1) / DMD_SLICES;
  const int r0 = lo + sl * per, r1 = r0 + per < hi ? r0 + per : hi;
  float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  // eight rows requested together (their additions keep the row order): one at a time, the chain of
  // three dependent loads per row took 27 us for 34 MB, now 17
  constexpr int RB = 8;
  for (int rb = r0; rb < r1; rb += RB) {
    int pair[RB];
    float w[RB];
    bf16x8_t a[RB], b[RB];
#pragma unroll
    for (int p = 0; p < RB; p++) pair[p] = pc.pair_of_row[rb + p < r1 ? rb + p : rb];
#pragma unroll
    for (int p = 0; p < RB; p++) {
      w[p] = pc.w[pair[p]];
      a[p] = *reinterpret_cast<const bf16x8_t *>(dy + (int64_t)(pair[p] / pc.k) * d + col);
      b[p] = *reinterpret_cast<const bf16x8_t *>(v + (int64_t)(rb + p < r1 ? rb + p : rb) * d + col);
    }
    __builtin_amdgcn_sched_barrier(0);   // or the loads sink into the additions' conditions
#pragma unroll
    for (int p = 0; p < RB; p++) {
      const bool valid = rb + p < r1;
#pragma unroll
      for (int i = 0; i < 8; i++) {
        const float t = fmaf(w[p] * (float)a[p][i], (float)b[p][i], acc[i]);
        acc[i] = valid ? t : acc[i];
      }
    }
  }
  float *o = part + ((int64_t)sl * pc.N + e) * d + col;
#pragma unroll
  for (int i = 0; i < 8; i++) o[i] = acc[i];
}

// per expert: dm [N, d]; shared magnitude: dm [d] = sum over the experts in ascending order
__global__ void dm_down_reduce_kernel(const float *__restrict__ part, const float *__restrict__ ninv,
                                      int N, int d, int shared, float *__restrict__ dm) {
  const int64_t n = (int64_t)N * d;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (shared ? d : n)) return;
  float tot = 0.f;
  for (int e = 0; e < (shared ? N : 1); e++) {
    const int64_t o = i + (int64_t)e * d;
    float acc = 0.f;
    for (int sl = 0; sl < DMD_SLICES; sl++) acc += part[(int64_t)sl * n + o];
    tot += acc * ninv[o];
  }
  dm[i] = tot;
}

size_t dm_down_part_floats(int N, int d) { return (size_t)DMD_SLICES * N * d; }

hipError_t launch_dm_down(const PairCtx &pc, int d, const void *dy, const void *v, const float *ninv,
                          float *part, float *dm, int shared, hipStream_t st) {
  hipLaunchKernelGGL(dm_down_part_kernel, dim3((d / 8 + 255) / 256, pc.N, DMD_SLICES), dim3(256), 0,
                     st, pc, d, (const bf16_t *)dy, (const bf16_t *)v, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t n = shared ? (int64_t)d : (int64_t)pc.N * d;
  hipLaunchKernelGGL(dm_down_reduce_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, part,
                     ninv, pc.N, d, shared, dm);
  return hipGetLastError();
}

// ---- magnitude gradients of gate / up from the fused stage's per-tile sums -----------------------
// dm[e, c] = ninv[e, c] * sum over the row tiles of expert e (ascending) of part[tile][c];
// blockIdx.z picks gate (0) or up (1).  The tiles of an expert are consecutive, 32 rows each.
// With a magnitude shared by the experts (grid y = 1, N experts walked here) dm[c] is the sum of
// the experts' terms in ascending order.
__global__ __launch_bounds__(256) void dm_tiles_reduce_kernel(
    const int32_t *__restrict__ offs, int f, int N, int shared, const float *__restrict__ part_g,
    const float *__restrict__ part_u, const float *__restrict__ ninv_g,
    const float *__restrict__ ninv_u, float *__restrict__ dm_g, float *__restrict__ dm_u) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= f) return;
  const float *part = blockIdx.z ? part_u : part_g;
  const float *ninv = blockIdx.z ? ninv_u : ninv_g;
  float *dm = blockIdx.z ? dm_u : dm_g;
  const int e_lo = shared ? 0 : blockIdx.y, e_hi = shared ? N : blockIdx.y + 1;
  int tile0 = 0;
  for (int q = 0; q < e_lo; q++) tile0 += (offs[q + 1] - offs[q] + 31) / 32;
  float tot = 0.f;
  for (int e = e_lo; e < e_hi; e++) {
    const int nt = (offs[e + 1] - offs[e] + 31) / 32;
    float acc = 0.f;
#pragma unroll 8
    for (int t = 0; t < nt; t++) acc += part[(int64_t)(tile0 + t) * f + c];
    tile0 += nt;
    tot += acc * ninv[(int64_t)e * f + c];
  }
  dm[shared ? c : (int64_t)e_lo * f + c] = tot;
}

hipError_t launch_dm_tiles_reduce(const int32_t *offs, int N, int f, const float *part_g,
                                  const float *part_u, const float *ninv_g, const float *ninv_u,
                                  float *dm_g, float *dm_u, int shared, hipStream_t st) {
  hipLaunchKernelGGL(dm_tiles_reduce_kernel, dim3((f + 255) / 256, shared ? 1 : N, 2), dim3(256), 0,
                     st, offs, f, N, shared, part_g, part_u, ninv_g, ninv_u, dm_g, dm_u);
  return hipGetLastError();
}

}  // namespace mixlora
