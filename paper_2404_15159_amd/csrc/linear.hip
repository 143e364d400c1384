// Plain LoRA linear (Eq. 1 with the scale alpha / r), the form the method puts on the attention
// projections (Section 3.2):  y = x W^T + s (x A^T) B^T  with W frozen.  Built from the same
// pieces as the feed-forward block.  bf16 with more than 128 rows, or more than four into fewer than
// 8192 columns: the rank-r projection s x A^T is made first (rank_project_kernel) and enters the
// frozen product as an extra K segment, in three bf16 pieces that hold all of its 24 bits.  Otherwise
// the frozen product and the projection share one GEMM launch and the rank-r update is added in place
// in fp32.  The gradients of A and B are outer-product sums over all tokens as one group.
#include "common.h"

#include <cmath>

using namespace mixlora;

namespace {

constexpr size_t ALIGN = 256;
inline size_t up(size_t v) { return (v + ALIGN - 1) / ALIGN * ALIGN; }
inline bool misaligned(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) != 0; }

inline int pad_rank(int r) { return (r + 7) & ~7; }

struct LinLayout {
  int rp;                         // rank entries the pass runs on: r rounded up to a multiple of 8
  size_t padA, padB, padgA, padgB;   // zero-padded copies of A, B (kept for the backward) and of dA, dB
  size_t P, P_T, tok_offs, ext, ext_B, gemm_part, fwd_end;
  size_t W_T, Bt, At, VB, VB_T, partials, bwd_end;
  size_t partial_floats, gemm_floats;
  int ldT;
  bool ext_fwd, ext_bwd;          // the rank-r term rides in the frozen product of that direction
};

LinLayout make_layout(const mixlora_linear_dims &D) {
  LinLayout L{};
  const size_t T = D.T, di = D.d_in, dn = D.d_out, r = pad_rank(D.r);
  const size_t E = D.dtype == MIXLORA_BF16 ? 2 : 4;
  const bool padded = (int)r != D.r;
  size_t o = 0;
  auto take = [&](size_t bytes) { size_t at = o; o = up(o + bytes); return at; };
  L.rp = (int)r;
  L.padA = take(padded ? r * di * E : 0);
  L.padB = take(padded ? dn * r * E : 0);
  L.P = take(T * r * 4);
  // Up to four rows are matrix-vector products; up to 128 rows into many columns stream the weights
  // through narrow tiles that take whole K tiles only (128 rows into 14336 columns 44 us that way, 56
  // with the extension).
  auto extends = [&](size_t cols) { return E == 2 && (T > 128 || (T > 4 && cols < 8192)); };
  L.ext_fwd = extends(dn);
  L.ext_bwd = extends(di);
  L.ldT = (int)((T + 15) / 16 * 16 + 16);
  L.P_T = take((size_t)L.ldT * r * 2);
  L.tok_offs = take(2 * 4);
  L.ext = take(L.ext_fwd || L.ext_bwd ? T * 3 * r * 2 : 0);
  {
    const size_t cf = L.ext_fwd ? dn : 0, cb = L.ext_bwd ? di : 0;
    L.ext_B = take((cf > cb ? cf : cb) * 3 * r * 2);
  }
  {   // partial tiles of products cut along K: at most one tile per CU
    const size_t slices = (di > dn ? di : dn) / 64 / 4;
    const size_t tiles = (T / 192 + 1) * ((di > dn ? di : dn) / 256 + 1) * slices;
    L.gemm_floats = (L.ext_fwd || L.ext_bwd) && slices >= 2 ? GEMM_SCRATCH_FLOATS / 256 * (tiles < 256 ? tiles : 256) : 0;
    L.gemm_part = take(L.gemm_floats * 4);
  }
  L.fwd_end = o;
  L.W_T = take(di * dn * E);
  L.Bt = take(r * dn * E);
  L.At = take(di * r * E);
  L.VB = take(T * r * 4);
  L.VB_T = take((size_t)L.ldT * r * 2);
  size_t pf = group_outer_mfma_partial_floats(1, (int)r, (int)di, (int)T, 2) +
              group_outer_mfma_partial_floats(1, (int)r, (int)dn, (int)T, 2);
  if (E == 4)
    pf = group_outer_partial_floats(1, (int)r, (int)di, (int)T) + group_outer_partial_floats(1, (int)r, (int)dn, (int)T);
  L.partial_floats = pf;
  L.partials = take(pf * 4);
  L.padgA = take(padded ? r * di * 4 : 0);
  L.padgB = take(padded ? dn * r * 4 : 0);
  L.bwd_end = o;
  return L;
}

int check_dims(const mixlora_linear_dims *D) {
  if (!D) return MIXLORA_E_NULL;
  if (D->dtype != MIXLORA_F32 && D->dtype != MIXLORA_BF16) return MIXLORA_E_DTYPE;
  if (D->T < 1 || D->d_in < 8 || D->d_out < 8 || D->r < 1 || D->r > 64) return MIXLORA_E_SHAPE;
  if (D->d_in % 8 || D->d_out % 8) return MIXLORA_E_SHAPE;
  if ((int64_t)D->T >= (1 << 24)) return MIXLORA_E_SHAPE;
  return MIXLORA_OK;
}

__global__ void set_pair_kernel(int32_t *p, int a, int b) {
  if (threadIdx.x == 0 && blockIdx.x == 0) { p[0] = a; p[1] = b; }
}

#define HIP_TRY(expr)                                   \
  do {                                                  \
    hipError_t e_ = (expr);                             \
    if (e_ != hipSuccess) return MIXLORA_E_HIP;         \
  } while (0)

GemmProblem problem(int M, int N, void *C, int64_t ldc, int c_f32, const void *A, int64_t lda,
                    const void *B, int64_t ldb, int K) {
  GemmProblem p{};
  p.M = M; p.N = N; p.C = C; p.ldc = ldc; p.c_f32 = c_f32; p.nseg = 1;
  p.seg[0].A = A; p.seg[0].lda = lda; p.seg[0].B = B; p.seg[0].ldb = ldb; p.seg[0].K = K;
  return p;
}

// P[t, q] = sum_c X[t, c] * Wq[q, c]  (r <= 64 columns), in three forms: fp32, transposed bf16 (the
// row factor of the gradient sums) and m * P (s = m 2^e, 1/2 <= |m| < 1) cut into three bf16 pieces by
// truncation, ext[t] = [hi(r) | mid(r) | lo(r)]: their sum is m * P to its last bit, and no piece
// overflows.  Trailing workgroups lay out the other factor of that term, Bx[c] = [B | B' | B'] 2^e with
// B' = B but zeros for infinities: hi alone meets those, or two pieces of opposite signs would make
// NaN of them.
// Bound by reading X once (33 MB at 4096 x 4096: 9 us); a workgroup owns 16 rows, its eight waves every
// eighth 128-column run of them, so that 256 workgroups have 2 waves per SIMD with 4 KB each in flight;
// fragments come straight from memory (whole 128-byte lines over four MFMA steps), Wq from the caches.
// The waves' sums are added in a fixed order.
template <int NQ>
__global__ __launch_bounds__(512) void rank_project_kernel(const bf16_t *__restrict__ X,
                                                           const bf16_t *__restrict__ Wq, int T, int K,
                                                           int r, float m, float *__restrict__ P,
                                                           bf16_t *__restrict__ PT, int ldT,
                                                           bf16_t *__restrict__ ext,
                                                           int32_t *__restrict__ tok_offs,
                                                           const bf16_t *__restrict__ Bm, int cols,
                                                           float b_scale, bf16_t *__restrict__ Bx) {
  __shared__ float red[8][NQ][64][4];
  const int row_blocks = (T + 15) >> 4;
  if ((int)blockIdx.x >= row_blocks) {   // workgroup-uniform; eight entries of a row of B per thread
    const int per = r >> 3, i = (blockIdx.x - row_blocks) * 512 + threadIdx.x;
    if (i >= cols * per) return;
    const int c = i / per, q0 = i % per * 8;
    bf16x8_t v = *reinterpret_cast<const bf16x8_t *>(Bm + (int64_t)c * r + q0), fin;
#pragma unroll
    for (int e = 0; e < 8; e++) {
      v[e] = (bf16_t)((float)v[e] * b_scale);
      fin[e] = __builtin_isinf((float)v[e]) ? (bf16_t)0.f : v[e];
    }
    bf16_t *o = Bx + (int64_t)c * 3 * r + q0;
    *reinterpret_cast<bf16x8_t *>(o) = v;
    *reinterpret_cast<bf16x8_t *>(o + r) = fin;
    *reinterpret_cast<bf16x8_t *>(o + 2 * r) = fin;
    return;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l15 = lane & 15, hi = lane >> 4;
  const int t0 = blockIdx.x * 16;
  if (blockIdx.x == 0 && threadIdx.x == 0) {   // all tokens are one group of the gradient sums
    tok_offs[0] = 0;
    tok_offs[1] = T;
  }
  const int row = t0 + l15 < T ? t0 + l15 : T - 1;
  const bf16_t *xr = X + (int64_t)row * K;
  const bf16_t *wr[NQ];
#pragma unroll
  for (int j = 0; j < NQ; j++) wr[j] = Wq + (int64_t)(j * 16 + l15 < r ? j * 16 + l15 : r - 1) * K;
  f32x4_t acc[NQ];
#pragma unroll
  for (int j = 0; j < NQ; j++) acc[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  for (int k0 = wave * 128; k0 < K; k0 += 8 * 128) {
    bf16x8_t fx[4], fw[NQ][4];
#pragma unroll
    for (int ks = 0; ks < 4; ks++) {
      const int k = k0 + ks * 32 + hi * 8;
      const int kc = k < K ? k : 0;
      fx[ks] = *reinterpret_cast<const bf16x8_t *>(xr + kc);
#pragma unroll
      for (int j = 0; j < NQ; j++) fw[j][ks] = *reinterpret_cast<const bf16x8_t *>(wr[j] + kc);
    }
#pragma unroll
    for (int ks = 0; ks < 4; ks++) {
      if (k0 + ks * 32 + hi * 8 >= K) {   // past the end: zeros on both sides
#pragma unroll
        for (int u = 0; u < 8; u++) fx[ks][u] = (bf16_t)0.f;
#pragma unroll
        for (int j = 0; j < NQ; j++)
#pragma unroll
          for (int u = 0; u < 8; u++) fw[j][ks][u] = (bf16_t)0.f;
      }
#pragma unroll
      for (int j = 0; j < NQ; j++)
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[j][ks], fx[ks], acc[j], 0, 0, 0);
    }
  }
#pragma unroll
  for (int j = 0; j < NQ; j++) *reinterpret_cast<f32x4_t *>(red[wave][j][lane]) = acc[j];
  __syncthreads();
  // acc[j][u] of lane (l15, hi): row l15, q = 16 j + 4 hi + u
  for (int i = threadIdx.x; i < NQ * 256; i += 512) {
    const int j = i >> 8, q = j * 16 + (i & 15), t = t0 + ((i >> 4) & 15);
    if (q >= r || t >= T) continue;
    const int ln = ((i >> 2) & 3) * 16 + ((i >> 4) & 15), u = i & 3;
    float v = red[0][j][ln][u];
#pragma unroll
    for (int w = 1; w < 8; w++) v += red[w][j][ln][u];
    P[(int64_t)t * r + q] = v;
    PT[(int64_t)q * ldT + t] = (bf16_t)v;
    const float mp = m * v;
    const bool finite = (__float_as_uint(mp) & 0x7f800000u) != 0x7f800000u;
    const float h = finite ? __uint_as_float(__float_as_uint(mp) & 0xffff0000u) : mp;
    const float rest = finite ? mp - h : 0.f;
    const float mid = __uint_as_float(__float_as_uint(rest) & 0xffff0000u);
    bf16_t *o = ext + (int64_t)t * 3 * r + q;
    o[0] = (bf16_t)h;
    o[r] = (bf16_t)mid;
    o[2 * r] = (bf16_t)(rest - mid);
  }
}

// C = X Wmain^T + s (X Wq^T) Wr^T where the rank-r term rides in the product: the projection, then one
// product over the K segments [X | hi mid lo] x [Wmain | Bx].  P and PT keep the projection (unscaled).
// Against the product beside an unextended projection, its slices' sum and an in-place update of C:
// 4096 x 4096 x 4096, rank 16, 157 -> 108 us, and one rounding of C less (projection 12.5 us of which the
// other factor's layout 1.5, product 109 and its one K tile for the term: two pieces in two segments of their
// own came to the same).
int extended_product(const LinLayout &L, char *ws, int T, int Nmain, int r, int K, float s, const void *X,
                     const void *Wmain, void *C, const void *Wq, const void *Wr, float *P, void *PT,
                     hipStream_t st) {
  int e = 0;   // s = m 2^e
  if (std::isfinite(s)) std::frexp(s, &e);
  e = e < -100 ? -100 : e > 100 ? 100 : e;
  const float m = std::ldexp(s, -e);
  const dim3 grid((T + 15) / 16 + (Nmain * (r / 8) + 511) / 512), block(512);
  const int slot = prof_on() ? prof_mark_begin(PROF_OTHER, st) : -1;
#define MIXLORA_RANKP(NQ_)                                                                          \
  hipLaunchKernelGGL(rank_project_kernel<NQ_>, grid, block, 0, st, (const bf16_t *)X,               \
                     (const bf16_t *)Wq, T, K, r, m, P, (bf16_t *)PT, L.ldT, (bf16_t *)(ws + L.ext), \
                     (int32_t *)(ws + L.tok_offs), (const bf16_t *)Wr, Nmain, std::ldexp(1.f, e),   \
                     (bf16_t *)(ws + L.ext_B))
  if (r <= 16) MIXLORA_RANKP(1);
  else if (r <= 32) MIXLORA_RANKP(2);
  else MIXLORA_RANKP(4);
#undef MIXLORA_RANKP
  if (slot >= 0) prof_mark_end(slot, st, 0.0);
  HIP_TRY(hipGetLastError());
  GemmProblem p = problem(T, Nmain, C, Nmain, 0, X, K, Wmain, K, K);
  p.seg[1] = GemmSeg{ws + L.ext, ws + L.ext_B, 3 * r, 3 * r, 3 * r};
  p.nseg = 2;
  HIP_TRY(launch_gemm(MIXLORA_BF16, &p, 1, st, GemmScratch{L.gemm_floats ? (float *)(ws + L.gemm_part) : nullptr, L.gemm_floats}));
  return MIXLORA_OK;
}

// C_main = X Wmain^T  (storage dtype)  and the rank-r projection  C_small = X Wsmall^T  (float32, r
// columns), one launch where both have a kernel in common.
int product_and_projection(int dtype, int T, int Nmain, int r, int K, const void *X, const void *Wmain,
                           void *Cmain, const void *Wsmall, float *Csmall, hipStream_t st) {
  const GemmProblem p[2] = {problem(T, Nmain, Cmain, Nmain, 0, X, K, Wmain, K, K),
                            problem(T, r, Csmall, r, 1, X, K, Wsmall, K, K)};
  HIP_TRY(launch_gemm(dtype, p, 2, st));
  return MIXLORA_OK;
}

}  // namespace

extern "C" {

size_t mixlora_lora_linear_workspace_bytes(const mixlora_linear_dims *dims, int for_backward) {
  if (check_dims(dims) != MIXLORA_OK) return 0;
  const LinLayout L = make_layout(*dims);
  return for_backward ? L.bwd_end : L.fwd_end;
}

int mixlora_lora_linear_forward(const mixlora_linear_dims *dims, const void *W, const void *A,
                                const void *B, const void *x, void *y, void *workspace,
                                size_t workspace_bytes, void *stream) {
  const int rc = check_dims(dims);
  if (rc) return rc;
  if (!W || !A || !B || !x || !y || !workspace) return MIXLORA_E_NULL;
  for (const void *p : {W, A, B, x, (const void *)y, (const void *)workspace})
    if (misaligned(p)) return MIXLORA_E_ALIGN;
  mixlora_linear_dims D = *dims;
  const LinLayout L = make_layout(D);
  if (workspace_bytes < L.fwd_end) return MIXLORA_E_WORKSPACE;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  char *ws = reinterpret_cast<char *>(workspace);
  if (L.rp != D.r) {   // run on zero-padded banks (they stay in the workspace for the backward)
    const RelayoutJob jobs[2] = {job_rank_resize(A, ws + L.padA, 1, D.r, L.rp, D.d_in, true),
                                 job_rank_resize(B, ws + L.padB, 1, D.r, L.rp, D.d_out, false)};
    HIP_TRY(launch_relayout(D.dtype, jobs, 2, st));
    A = ws + L.padA;
    B = ws + L.padB;
    D.r = L.rp;
  }
  if (L.ext_fwd)
    return extended_product(L, ws, D.T, D.d_out, D.r, D.d_in, D.lora_scale, x, W, y, A, B,
                            (float *)(ws + L.P), ws + L.P_T, st);
  // y0 = x W^T and P = x A^T in one launch (both read x), then y = y0 + s P B^T in place
  const int grc = product_and_projection(D.dtype, D.T, D.d_out, D.r, D.d_in, x, W, y, A,
                                         (float *)(ws + L.P), st);
  if (grc) return grc;
  HIP_TRY(launch_lowrank_add(D.dtype, y, (const float *)(ws + L.P), B, D.T, D.d_out, D.r,
                             D.lora_scale, st));
  return MIXLORA_OK;
}

int mixlora_lora_linear_backward(const mixlora_linear_dims *dims, const void *W, const void *W_T,
                                 const void *A, const void *B, const void *x, const void *dy,
                                 void *workspace, size_t workspace_bytes, void *dx, float *dA,
                                 float *dB, void *stream) {
  const int rc = check_dims(dims);
  if (rc) return rc;
  if (!W || !A || !B || !x || !dy || !workspace || !dx || !dA || !dB) return MIXLORA_E_NULL;
  for (const void *p : {W, A, B, x, dy, (const void *)workspace, (const void *)dx, (const void *)dA,
                        (const void *)dB})
    if (misaligned(p)) return MIXLORA_E_ALIGN;
  if (W_T && misaligned(W_T)) return MIXLORA_E_ALIGN;
  const mixlora_linear_dims &D = *dims;
  const LinLayout L = make_layout(D);
  if (workspace_bytes < L.bwd_end) return MIXLORA_E_WORKSPACE;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  char *ws = reinterpret_cast<char *>(workspace);
  const int T = D.T, di = D.d_in, dn = D.d_out, r = L.rp, dt = D.dtype;
  float *dA_user = dA, *dB_user = dB;
  if (L.rp != D.r) {   // padded banks from the forward pass; padded gradients, cut back at the end
    A = ws + L.padA;
    B = ws + L.padB;
    dA = (float *)(ws + L.padgA);
    dB = (float *)(ws + L.padgB);
  }
  const float s = D.lora_scale;
  if (!W_T) {
    HIP_TRY(launch_transpose(dt, W, ws + L.W_T, dn, di, st));
    W_T = ws + L.W_T;
  }
  {
    const RelayoutJob jobs[2] = {job_bank_T(B, 1, dn, r, ws + L.Bt),     // [d_out, r] -> [r, d_out]
                                 job_bank_T(A, 1, r, di, ws + L.At)};    // [r, d_in]  -> [d_in, r]
    HIP_TRY(launch_relayout(dt, jobs, 2, st));
  }
  if (L.ext_bwd) {
    const int erc = extended_product(L, ws, T, di, r, dn, s, dy, W_T, dx, ws + L.Bt, ws + L.At,
                                     (float *)(ws + L.VB), ws + L.VB_T, st);
    if (erc) return erc;
  } else {
    hipLaunchKernelGGL(set_pair_kernel, dim3(1), dim3(64), 0, st, (int32_t *)(ws + L.tok_offs), 0, T);
    HIP_TRY(hipGetLastError());
    // dx0 = dy W and VB = dy B in one launch (both read dy), then dx = dx0 + s VB A in place
    const int grc = product_and_projection(dt, T, di, r, dn, dy, W_T, dx, ws + L.Bt,
                                           (float *)(ws + L.VB), st);
    if (grc) return grc;
    HIP_TRY(launch_lowrank_add(dt, dx, (const float *)(ws + L.VB), ws + L.At, T, di, r, s, st));
    if (dt == MIXLORA_BF16)
      HIP_TRY(launch_f32_to_bf16T((const float *)(ws + L.VB), T, r, ws + L.VB_T, L.ldT, st));
  }
  if (dt == MIXLORA_BF16 && !L.ext_fwd)   // else the forward's projection kernel has written it
    HIP_TRY(launch_f32_to_bf16T((const float *)(ws + L.P), T, r, ws + L.P_T, L.ldT, st));
  // dA = s VB^T x  [r, d_in];  dB = s dy^T P  [d_out, r]: outer-product sums over all tokens
  const int32_t *tok = (const int32_t *)(ws + L.tok_offs);
  float *part = (float *)(ws + L.partials);
  if (dt == MIXLORA_BF16) {
    const GomJob go[2] = {GomJob{ws + L.VB_T, x, dA, tok, nullptr, 1, r, di, 1, T, L.ldT, 2, 1, s},
                          GomJob{ws + L.P_T, dy, dB, tok, nullptr, 1, r, dn, 1, T, L.ldT, 2, 0, s}};
    HIP_TRY(launch_group_outer_mfma(go, 2, part, L.partial_floats, st));
  } else {
    const GoJob go[2] = {
        GoJob{tok, nullptr, (const float *)(ws + L.VB), (const float *)x, dA, 1, r, di, 1, T, 1, s},
        GoJob{tok, nullptr, (const float *)(ws + L.P), (const float *)dy, dB, 1, r, dn, 1, T, 0, s}};
    HIP_TRY(launch_group_outer(go, 2, part, L.partial_floats, st));
  }
  if (L.rp != D.r) {
    const RelayoutJob jobs[2] = {job_rank_resize(dA, dA_user, 1, L.rp, D.r, di, true),
                                 job_rank_resize(dB, dB_user, 1, L.rp, D.r, dn, false)};
    HIP_TRY(launch_relayout(MIXLORA_F32, jobs, 2, st));
  }
  return MIXLORA_OK;
}

}  // extern "C"
