// Per-pair stages (Algorithm 1 lines 11-15 and their backward) on token tiles whose tokens all
// share one unordered pair of experts {a, b} (top-2 routing, bf16, MFMA).
//
// The grouped stages of csrc/fused.hip work on rows grouped by expert: a token's two pairs fall
// into different tiles, so the shared projections G, U of a token are read twice and the weighted
// combination of its two pairs (Eq. 6, moved in front of the linear frozen down projection) needs
// another pass over the grouped rows.  Here the TOKENS are grouped by their unordered expert pair
// instead (csrc/router.hip), 32 tokens of one group to a tile.
//
// Both kernels put G and U (and H) through LDS row-major into the accumulators' layout and add the experts'
// rank-r deltas there by MFMA: no delta is rounded, and the element math (13 -> 9 vector instructions per
// pair and column in the forward) works on a lane's 16 columns of one row.  A lane reads its own columns and unpacks
// them; as a product with the identity that is 10-15 % fewer vector instructions and the same time (step at the 7B
// shape 2047 us, read 2044), but a non-finite element then makes NaN of the 31 columns beside it.  (As it is, it
// reaches its own column and what is formed from its whole row.)
// What bounds them is memory (the forward moves 4.4 TB/s, the copy rate being 5.1) and, in the backward, the
// latency of its chain of phases at two wavefronts per SIMD; so what is left to gain is bytes: the backward
// makes the gradient sums of its three d_ff-wide operands itself, and neither the activations nor dg and du of a
// pair are ever stored.  4096 tokens at the 7B shape, us, against the two kernels that stored all three: forward 135 ->
// 91, backward 268 -> 258 + 26 for adding its partial sums, gradient sums 150 -> 65; the step 2146 -> 2055.
// 16384 tokens of the L3-8B shape: 529 -> 337, 1162 -> 1363 + 38, 855 -> 271; 10716 -> 10340.
//
// LDS tiles are those of csrc/fused.hip.
#include "fused_common.h"

namespace mixlora {

// Uniform base + 32-bit BYTE offset: the form the hardware addresses with a scalar base and one
// vector register, so the loop carries no 64-bit address arithmetic.
__device__ __forceinline__ bf16x8_t ldg8(const bf16_t *base, uint32_t byte_off) {
  return *reinterpret_cast<const bf16x8_t *>(reinterpret_cast<const char *>(base) + byte_off);
}
__device__ __forceinline__ void stg8(bf16_t *base, uint32_t byte_off, const bf16x8_t &v) {
  *reinterpret_cast<bf16x8_t *>(reinterpret_cast<char *>(base) + byte_off) = v;
}

static_assert(PG_TILE_ROWS == FT_ROWS, "the grouping kernel cuts tiles of FT_ROWS tokens");

// Forward.  Per pair: Q_part[split][row(t, j)][q]; per token:
// a_comb[t, :] = w_ta a_ta + w_tb a_tb (the lower-numbered expert's term first, fp32, one rounding).
//
// One wavefront owns a 32-token x 64-column piece for BOTH experts of the tile: G and U are fetched once, the two
// activations stay in registers until their weighted sum is formed.  Wavefronts never wait for each other
// inside the loop.  Offsets into the [T, f] / [2T, f] arrays are 32-bit (host check).
__global__ __launch_bounds__(FT_WAVES * 64, 2) void swiglu_fwd_pg_kernel(
    PairCtx pc, int f, float s, const int32_t *__restrict__ tok_of_pos,
    const int32_t *__restrict__ tile_info, const int32_t *__restrict__ ntiles,
    const bf16_t *__restrict__ G, const bf16_t *__restrict__ U, const float *__restrict__ Pg_all,
    const float *__restrict__ Pu_all, const bf16_t *__restrict__ B_gate,
    const bf16_t *__restrict__ B_up, const bf16_t *__restrict__ A_down,
    bf16_t *__restrict__ a_comb, float *__restrict__ Q_part, int nsplit) {
  constexpr int TILES = 3;   // per wavefront: G then expert a's activations, U then expert b's, the combination
  __shared__ __align__(16) bf16_t lds[FT_WAVES * TILES * FT_TILE];
  __shared__ int growmap[2][FT_ROWS];   // expert-grouped row of every tile row, per expert
  if ((int)blockIdx.x >= ntiles[0]) return;
  const int32_t *ti = tile_info + (int64_t)blockIdx.x * 4;
  const int r = pc.r, R = pc.N * r, nP = pc.T * 2;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l31 = lane & 31, hi = lane >> 5, rr = lane >> 3, cc = lane & 7;
  const int gid = ti[0], row0 = ti[1], rows = ti[2];
  const int ex[2] = {gid / pc.N, gid % pc.N};
  bf16_t *tiles = lds + wave * TILES * FT_TILE;
  const int q0 = hi * 8;
  const bool q_in = q0 < r;   // r <= 16: one MFMA step over the rank

  // MFMA role: second-operand fragments of this lane's row (token), per expert
  bf16x8_t pg[2], pu[2];
  {
    const int64_t tm = tok_of_pos[row0 + (l31 < rows ? l31 : 0)];
#pragma unroll
    for (int x = 0; x < 2; x++) {
      const int64_t o = tm * R + ex[x] * r + (q_in ? q0 : 0);
      pg[x] = cvt8(Pg_all + o, q_in, s);
      pu[x] = cvt8(Pu_all + o, q_in, s);
    }
  }
  // row-major role: the four rows (8p + rr) this lane serves
  uint32_t gsrc[4];
  bool rvalid[4];
#pragma unroll
  for (int p = 0; p < 4; p++) {
    const int rl = 8 * p + rr;
    rvalid[p] = rl < rows;
    const int64_t tok = tok_of_pos[row0 + (rvalid[p] ? rl : 0)];
    gsrc[p] = (uint32_t)(tok * f) * 2u;   // bytes
  }
  // MFMA result role: this lane's row's routing weights, and its grouped row with expert hi
  float wx[2];
  int grow;
  {
    const int64_t tok = tok_of_pos[row0 + (l31 < rows ? l31 : 0)];
    const int slot_a = pc.idx[tok * 2] == ex[0] ? 0 : 1;   // expert a's slot of this token
    wx[0] = pc.w[tok * 2 + slot_a];
    wx[1] = pc.w[tok * 2 + (slot_a ^ 1)];
    grow = pc.row_of_pair[tok * 2 + (slot_a ^ hi)];
  }
  f32x16_t accq[2];
#pragma unroll
  for (int x = 0; x < 2; x++)
#pragma unroll
    for (int i = 0; i < 16; i++) accq[x][i] = 0.f;

  const int nsb = (f + FT_SB - 1) / FT_SB;
  const int per = (nsb + nsplit - 1) / nsplit;
  const int sb_lo = blockIdx.y * per;
  const int sb_hi = sb_lo + per < nsb ? sb_lo + per : nsb;
  const bf16_t *bg_e[2], *bu_e[2], *ad_e[2];
#pragma unroll
  for (int x = 0; x < 2; x++) {
    bg_e[x] = B_gate + (int64_t)ex[x] * f * r;
    bu_e[x] = B_up + (int64_t)ex[x] * f * r;
    ad_e[x] = A_down + (int64_t)ex[x] * r * f;
  }

  bf16x8_t wg[2][2], wu[2][2], wf[2][4], gnx[4], unx[4];
  auto load_w = [&](int c0) {
#pragma unroll
    for (int b = 0; b < 2; b++) {
      int col = c0 + 32 * b + l31;
      col = col < f ? col : f - 1;
      const uint32_t o = ((uint32_t)col * (uint32_t)r + (q_in ? q0 : 0)) * 2u;
#pragma unroll
      for (int x = 0; x < 2; x++) {
        wg[x][b] = ldg8(bg_e[x], o);
        wu[x][b] = ldg8(bu_e[x], o);
      }
    }
  };
  auto load_wf = [&](int c0) {
#pragma unroll
    for (int s4 = 0; s4 < 4; s4++) {
      int col = c0 + 16 * s4 + 8 * hi;
      col = col < f ? col : f - 8;
      const uint32_t o = ((uint32_t)(l31 < r ? l31 : 0) * (uint32_t)f + col) * 2u;
#pragma unroll
      for (int x = 0; x < 2; x++) wf[x][s4] = ldg8(ad_e[x], o);
    }
  };
  auto col_of = [&](int c0) { const int c = c0 + 8 * cc; return (uint32_t)(c < f ? c : f - 8) * 2u; };   // bytes
  if (sb_lo + wave < sb_hi) {
    const int cf = (sb_lo + wave) * FT_SB;
    load_w(cf);
#pragma unroll
    for (int p = 0; p < 4; p++) {
      gnx[p] = ldg8(G, gsrc[p] + col_of(cf));
      unx[p] = ldg8(U, gsrc[p] + col_of(cf));
    }
    load_wf(cf);
  }
  growmap[hi][l31] = grow;   // every wavefront the same (under a condition the load waits for its turn there)
  for (int sb = sb_lo + wave; sb < sb_hi; sb += FT_WAVES) {
    const int c0 = sb * FT_SB;
    const int cn = sb + FT_WAVES < sb_hi ? c0 + FT_WAVES * FT_SB : c0;   // next (or again this)
    const bool tail = c0 + FT_SB > f;
    const uint32_t col = (c0 + 8 * cc) * 2u;   // bytes
    const bool cvalid = c0 + 8 * cc < f;
#pragma unroll
    for (int p = 0; p < 4; p++) {
      const int toff = (8 * p + rr) * FT_PITCH + 8 * cc;
      *reinterpret_cast<bf16x8_t *>(tiles + toff) = gnx[p];
      *reinterpret_cast<bf16x8_t *>(tiles + FT_TILE + toff) = unx[p];
    }
    __builtin_amdgcn_wave_barrier();
    // the next piece's shared projections, a whole piece before they are needed
#pragma unroll
    for (int p = 0; p < 4; p++) {
      gnx[p] = ldg8(G, gsrc[p] + col_of(cn));
      unx[p] = ldg8(U, gsrc[p] + col_of(cn));
    }
#pragma unroll
    for (int b = 0; b < 2; b++) {
      // (block b overwrites its own columns only)
      const f32x16_t g0 = tile_get(tiles, l31, hi, 32 * b), u0 = tile_get(tiles + FT_TILE, l31, hi, 32 * b);
      f32x16_t comb;
#pragma unroll
      for (int x = 0; x < 2; x++) {
        f32x16_t g = g0, u = u0;   // + the expert's rank-r deltas
        g = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wg[x][b], pg[x], g, 0, 0, 0);
        u = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wu[x][b], pu[x], u, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 16; i++) {
          g[i] = g[i] * fsigmoid(g[i]) * u[i];   // columns past f: finite, meet zeroed weights
          comb[i] = x == 0 ? wx[0] * g[i] : fmaf(wx[1], g[i], comb[i]);
        }
        tile_put(tiles + x * FT_TILE, l31, hi, 32 * b, g);
      }
      tile_put(tiles + 2 * FT_TILE, l31, hi, 32 * b, comb);
      __builtin_amdgcn_sched_barrier(0);   // (interleaved, the blocks run out of registers)
    }
    load_w(cn);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int p = 0; p < 4; p++) {
      const bf16_t *tp = tiles + (8 * p + rr) * FT_PITCH + 8 * cc;
      if (rvalid[p] && cvalid) stg8(a_comb, gsrc[p] + col, ld8(tp + 2 * FT_TILE));
    }
    // Q_x += a_x[rows, 64 cols] * A_down[e_x, q, same cols]^T : four K steps of 16 columns
#pragma unroll
    for (int s4 = 0; s4 < 4; s4++) {
      const bool zero_w = tail && c0 + 16 * s4 + 8 * hi >= f;
#pragma unroll
      for (int x = 0; x < 2; x++) {
        const bf16x8_t af = ld8(tiles + x * FT_TILE + l31 * FT_PITCH + 16 * s4 + 8 * hi);
        bf16x8_t w = wf[x][s4];
        if (zero_w) w = zero8();
        accq[x] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af, w, accq[x], 0, 0, 0);
      }
    }
    load_wf(cn);
    __builtin_amdgcn_wave_barrier();
  }
  // accq[x][i]: row 8*(i/4) + 4*hi + i%4 of the tile, q = l31.  Each wavefront parks its
  // sums in its own (now dead) tile space; then the four are added in a fixed order.
  static_assert(sizeof(float) * 2 * 16 * 64 <= sizeof(bf16_t) * TILES * FT_TILE, "reduction space");
  float *mine = reinterpret_cast<float *>(tiles);
#pragma unroll
  for (int x = 0; x < 2; x++)
#pragma unroll
    for (int i = 0; i < 16; i++) mine[(x * 16 + i) * 64 + lane] = accq[x][i];
  __syncthreads();
  const int wstride = TILES * FT_TILE / 2;   // floats between two wavefronts' spaces
  const float *base = reinterpret_cast<const float *>(lds);
  for (int idx2 = threadIdx.x; idx2 < 2 * 16 * 64; idx2 += FT_WAVES * 64) {
    const int x = idx2 / (16 * 64), i = (idx2 / 64) % 16, ln = idx2 % 64;
    const int q = ln & 31;
    const int rl = 8 * (i >> 2) + 4 * (ln >> 5) + (i & 3);
    if (q < r && rl < rows) {
      const float v = (base[idx2] + base[wstride + idx2]) + (base[2 * wstride + idx2] + base[3 * wstride + idx2]);
      Q_part[((int64_t)blockIdx.y * nP + growmap[x][rl]) * r + q] = v;
    }
  }
}

// Backward of the stage above on the same token tiles, with the three gradient sums over d_ff-wide operands
// (dB_gate, dB_up, dA_down) in it: the per-pair gradients dg, du and the activations they need never leave
// the workgroup.
//
// A workgroup owns 128 columns (PGB_COLS) and walks a run of consecutive tiles: wavefronts 0 and 1 ("role A")
// take the rows as rows of expert a, 64 columns each, wavefronts 2 and 3 ("role B") as rows of expert b.  The columns'
// bank rows stay in registers while the expert stays; the sums accumulate there (48 registers) and are
// flushed to the wavefront's own slot of the expert when it changes, which tiles ordered by expert pair
// make rare.  With H[t] = W_down^T dy[t]:
//   da = w H + A_down^T (w s VB),  dg = da * u * SiLU'(g),  du = da * SiLU(g),  dw += <H, a>
// in the accumulators' layout (a lane holds 16 columns of one row): G, U, H go through LDS row-major, the
// rank-r terms are added to them by MFMA, so no delta is rounded.  The results return to the tiles in LDS,
// rounded to bf16, where
//   - the two roles add each other's to their own and store the per-token sums, role A those of dg, role B of du,
//   - the rank-r products with B_gate^T, B_up^T (contraction over columns) read them by rows, and
//   - the gradient sums (contraction over rows) read them transposed (ds_read_b64_tr_b16).
// Rank-r products of a role's wavefronts are added through LDS, one partial sum per PGB_COLS columns.
constexpr int PGB_CW = 2, PGB_WAVES = 2 * PGB_CW, PGB_COLS = PGB_CW * FT_SB;   // PGB_CW: wavefronts of a role
typedef short s16x4_t __attribute__((ext_vector_type(4)));

struct PgBwd {
  PairCtx pc;
  int f, nwg;
  float s;
  const int32_t *tok_of_pos, *tile_info, *ntiles;
  const bf16_t *G, *U, *H;
  const float *Pg_all, *Pu_all, *VB_all;
  const bf16_t *B_gate, *B_up, *AdT, *BgT, *BuT;
  bf16_t *dgsum, *dusum;
  float *dw_part, *T_part;   // [row][column block]; [2][column block][row][r]
  float *slots;              // [workgroup + column block][wavefront][expert][3][r][64]: along the items one of the two grows
  uint32_t *masks;           // [workgroup + column block][wavefront]: experts whose slot is in use
};

// run of workgroup wg: items (column block, tile), tiles fastest; at most two column blocks (nwg >= blocks)
__device__ __forceinline__ int pgb_run(int nt, int ncb, int nwg) { return (nt * ncb + nwg - 1) / nwg; }

// four rows of one column per lane: rows 4 hi .. 4 hi + 3 of the 16 columns at p, as MFMA operand elements
__device__ __forceinline__ s16x4_t ld4_t(const bf16_t *p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) s16x4_t *)(__attribute__((address_space(3))) const bf16_t *)p);
}
__device__ __forceinline__ bf16x8_t ld8_t(const bf16_t *p, int pitch) {   // rows 4 hi + .. and 16 + 4 hi + ..
  typedef short s16x8_t __attribute__((ext_vector_type(8)));
  const s16x4_t a = ld4_t(p), b = ld4_t(p + 16 * pitch);
  const s16x8_t v = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8_t, v);
}

struct PgbShared {
  bf16_t tile[PGB_WAVES][3][FT_TILE];
  float T[PGB_WAVES][2][FT_ROWS][16];
  bf16_t P[2][3][FT_ROWS][16];
  int grow[2][2][FT_ROWS], tok[FT_ROWS];
  float dw[PGB_WAVES][FT_ROWS];
};

__global__ __launch_bounds__(PGB_WAVES * 64, 2) void swiglu_bwd_pg_kernel(PgBwd a) {
  extern __shared__ __align__(16) unsigned char lds[];
  PgbShared &sh = *reinterpret_cast<PgbShared *>(lds);
  const PairCtx &pc = a.pc;
  const int f = a.f, r = pc.r, N = pc.N, R = N * r, nP = pc.T * 2;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int role = wave / PGB_CW, cw = wave % PGB_CW;
  const int l31 = lane & 31, hi = lane >> 5, rr = lane >> 3, cc = lane & 7, l15 = lane & 15, h4 = lane >> 4;
  const int nt = a.ntiles[0], ncb = (f + PGB_COLS - 1) / PGB_COLS, per = pgb_run(nt, ncb, a.nwg);
  // consecutive runs on one XCD (workgroups are dealt to the eight in turn): its L2 serves the banks of an eighth of
  // the columns, and the row factors to all of these
  const int xq = a.nwg >> 3, xrem = a.nwg & 7, xcd = blockIdx.x & 7;
  const int wgid = xcd * xq + (xcd < xrem ? xcd : xrem) + (blockIdx.x >> 3);
  const int i0 = wgid * per, i1 = i0 + per < nt * ncb ? i0 + per : nt * ncb;
  if (i0 >= i1) return;
  bf16_t *t0 = sh.tile[wave][0], *t1 = sh.tile[wave][1], *t2 = sh.tile[wave][2];
  // ---- this wavefront's banks and sums for one (expert, column block)
  bf16x8_t wg[2], wu[2], wd[2], tw[2][2];
  f32x4_t dacc[3][4];
  uint32_t used[2] = {0, 0};
  int e = -1, cb = -1;
  const int cb_first = i0 / nt;
  auto flush = [&]() {
    const int hf = cb - cb_first;
    float *dst = a.slots + (((size_t)(wgid + cb) * PGB_WAVES + wave) * N + e) * 3 * r * 64;
    const bool again = (used[hf] >> e) & 1;
    if (l15 < r) {
#pragma unroll
      for (int q = 0; q < 3; q++)
#pragma unroll
        for (int j = 0; j < 4; j++) {
          f32x4_t *p = reinterpret_cast<f32x4_t *>(dst + (q * r + l15) * 64 + 16 * j + 4 * h4);
          *p = again ? *p + dacc[q][j] : dacc[q][j];
        }
    }
    used[hf] |= 1u << e;
  };
  auto begin = [&](int c0) {   // (columns past f: clamped loads, zero weights of the products over columns)
    const bf16_t *bg_e = a.B_gate + (int64_t)e * f * r, *bu_e = a.B_up + (int64_t)e * f * r;
    const bf16_t *ad_e = a.AdT + (int64_t)e * f * r;
    const bf16_t *bt_e[2] = {a.BgT + (int64_t)e * r * f, a.BuT + (int64_t)e * r * f};
    const int q0 = 8 * hi < r ? 8 * hi : 0;   // (past r the row factors are zero)
#pragma unroll
    for (int b = 0; b < 2; b++) {
      int col = c0 + 32 * b + l31;
      col = col < f ? col : f - 1;
      const uint32_t o = ((uint32_t)col * (uint32_t)r + q0) * 2u;
      wg[b] = ldg8(bg_e, o);
      wu[b] = ldg8(bu_e, o);
      wd[b] = ldg8(ad_e, o);
    }
#pragma unroll
    for (int bank = 0; bank < 2; bank++)
#pragma unroll
      for (int ks = 0; ks < 2; ks++) {
        const int col = c0 + 32 * ks + 8 * h4;
        tw[bank][ks] = ldg8(bt_e[bank], ((uint32_t)(l15 < r ? l15 : 0) * (uint32_t)f + (col < f ? col : f - 8)) * 2u);
        if (col >= f) tw[bank][ks] = zero8();
      }
#pragma unroll
    for (int q = 0; q < 3; q++)
#pragma unroll
      for (int j = 0; j < 4; j++) dacc[q][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  };

  // ---- what a tile needs from memory: requested one tile ahead, its tokens two, its place three, and
  // nothing loaded is looked at in the iteration that asks for it
  bf16x8_t gn[4], un[4], hn[4];
  float4 pf[3][2];                     // fp32 rank entries 8 hi .. of row l31: Pg, Pu, VB
  float2 w2;                           // row l31: routing weights, grouped rows and expert of its two slots
  int2 grow2;
  int idx0;
  int tokp[4], tokm, tokl;             // tokens of the rows 8 p + rr and of row l31 (tokl: that of w2 ..)
  int32_t inf[3];                      // {group, first position, rows}
  auto clampi = [&](int i) { return i < i1 ? i : i1 - 1; };
  auto place = [&](int i) {
    const int32_t *ti = a.tile_info + (int64_t)(clampi(i) % nt) * 4;
    inf[0] = ti[0];
    inf[1] = ti[1];
    inf[2] = ti[2];
  };
  auto tokens = [&](int r0, int n) {
#pragma unroll
    for (int p = 0; p < 4; p++) tokp[p] = a.tok_of_pos[r0 + (8 * p + rr < n ? 8 * p + rr : 0)];
    tokm = a.tok_of_pos[r0 + (l31 < n ? l31 : 0)];
  };
  auto request = [&](int c0) {   // from tokp
#pragma unroll
    for (int p = 0; p < 4; p++) {
      const int c = c0 + 8 * cc;
      const uint32_t o = ((uint32_t)tokp[p] * (uint32_t)f + (c < f ? c : f - 8)) * 2u;
      gn[p] = ldg8(a.G, o);
      un[p] = ldg8(a.U, o);
      hn[p] = ldg8(a.H, o);
    }
  };
  auto request_rows = [&](int ex, int tok) {   // tok: token of row l31
    const int64_t o = (int64_t)tok * R + ex * r + (8 * hi < r ? 8 * hi : 0);
    const float *src[3] = {a.Pg_all + o, a.Pu_all + o, a.VB_all + o};
#pragma unroll
    for (int q = 0; q < 3; q++) {
      pf[q][0] = *reinterpret_cast<const float4 *>(src[q]);
      pf[q][1] = *reinterpret_cast<const float4 *>(src[q] + 4);
    }
    tokl = tok;
    w2 = *reinterpret_cast<const float2 *>(pc.w + (int64_t)tok * 2);
    grow2 = *reinterpret_cast<const int2 *>(pc.row_of_pair + (int64_t)tok * 2);
    idx0 = pc.idx[(int64_t)tok * 2];
  };
  auto cvt = [&](const float4 (&v)[2], float scale, bool valid) {
    bf16x8_t o;
    const float x[8] = {v[0].x, v[0].y, v[0].z, v[0].w, v[1].x, v[1].y, v[1].z, v[1].w};
#pragma unroll
    for (int m = 0; m < 8; m++) o[m] = (bf16_t)(valid ? x[m] * scale : 0.f);
    return o;
  };
  auto expert_of = [&](int g) { return role ? g % N : g / N; };
  auto col_of = [&](int block) { return block * PGB_COLS + cw * FT_SB; };
  // banks and sums for the tile to come
  auto change = [&](int ex, int block) {
    if (col_of(block) >= f || (ex == e && block == cb)) return;
    if (e >= 0) flush();
    e = ex;
    cb = block;
    begin(col_of(block));
  };

  int gid, rows, gid1, rows1, gid2, row02, rows2;   // tiles i, i + 1, i + 2
  auto take = [&](int &g, int &r0, int &n) {
    g = __builtin_amdgcn_readfirstlane(inf[0]);
    r0 = __builtin_amdgcn_readfirstlane(inf[1]);
    n = __builtin_amdgcn_readfirstlane(inf[2]);
  };
  place(i0);
  {
    int row0;
    take(gid, row0, rows);
    tokens(row0, rows);
  }
  request(col_of(cb_first));
  request_rows(expert_of(gid), tokm);
  change(expert_of(gid), cb_first);
  place(i0 + 1);
  {
    int row0;
    take(gid1, row0, rows1);
    tokens(row0, rows1);
  }
  place(i0 + 2);
  int last_rows = 0, last_cb = 0;
  auto add_waves = [&](int par) {      // rank-r products and <H, a> of the tile before, summed over its column wavefronts
    const int left = (f - last_cb * PGB_COLS + FT_SB - 1) / FT_SB, live = left < PGB_CW ? left : PGB_CW;
    const int tr = threadIdx.x % (PGB_CW * 64), w0 = role * PGB_CW;
#pragma unroll
    for (int x = 0; x < 256 / (PGB_CW * 64); x++) {   // four rank entries of a row each
      const int at = tr + x * PGB_CW * 64, bank = at >> 7, row = (at >> 2) & 31, q = (at & 3) * 4;
      if (row >= last_rows || q >= r) continue;
      f32x4_t v = *reinterpret_cast<const f32x4_t *>(&sh.T[w0][bank][row][q]);
      for (int w = 1; w < live; w++) v += *reinterpret_cast<const f32x4_t *>(&sh.T[w0 + w][bank][row][q]);
      *reinterpret_cast<f32x4_t *>(a.T_part + (((int64_t)bank * ncb + last_cb) * nP + sh.grow[par][role][row]) * r + q) = v;
    }
    if (tr < last_rows) {
      float v = sh.dw[w0][tr];
      for (int w = 1; w < live; w++) v += sh.dw[w0 + w][tr];
      a.dw_part[(int64_t)sh.grow[par][role][tr] * ncb + last_cb] = v;
    }
  };

  for (int i = i0; i < i1; i++) {
    const int par = i & 1, cbi = i / nt, ei = expert_of(gid), c0 = col_of(cbi);
    const bool live = c0 < f;          // wave-uniform, the same for both roles of a column
    if (i > i0) add_waves(par ^ 1);
    const bool q_in = 8 * hi < r;
    const int n = rows, slot = idx0 == ei ? 0 : 1;
    const float wm = slot ? w2.y : w2.x;
    if (live) {
#pragma unroll
      for (int p = 0; p < 4; p++) {
        const int o = (8 * p + rr) * FT_PITCH + 8 * cc;
        *reinterpret_cast<bf16x8_t *>(t0 + o) = gn[p];
        *reinterpret_cast<bf16x8_t *>(t1 + o) = un[p];
        *reinterpret_cast<bf16x8_t *>(t2 + o) = hn[p];
      }
    }
    const bf16x8_t pg = cvt(pf[0], a.s, q_in), pu = cvt(pf[1], a.s, q_in), vb = cvt(pf[2], wm * a.s, q_in);
    if (cw == 0) {   // the row factors of the sums, zero past the tile's rows; the grouped rows
      const bool in = q_in && l31 < n;
      *reinterpret_cast<bf16x8_t *>(&sh.P[role][0][l31][8 * hi]) = cvt(pf[0], 1.f, in);
      *reinterpret_cast<bf16x8_t *>(&sh.P[role][1][l31][8 * hi]) = cvt(pf[1], 1.f, in);
      *reinterpret_cast<bf16x8_t *>(&sh.P[role][2][l31][8 * hi]) = cvt(pf[2], wm, in);
      if (hi == 0) {
        sh.grow[par][role][l31] = slot ? grow2.y : grow2.x;
        if (role == 0) sh.tok[l31] = tokl;
      }
    }
    if (live) {
      float dw = 0.f;
#pragma unroll
      for (int b = 0; b < 2; b++) {
        f32x16_t g = tile_get(t0, l31, hi, 32 * b), u = tile_get(t1, l31, hi, 32 * b);
        const f32x16_t h = tile_get(t2, l31, hi, 32 * b);
        g = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wg[b], pg, g, 0, 0, 0);
        u = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wu[b], pu, u, 0, 0, 0);
        f32x16_t da;
#pragma unroll
        for (int x = 0; x < 16; x++) da[x] = wm * h[x];
        da = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wd[b], vb, da, 0, 0, 0);
#pragma unroll
        for (int x = 0; x < 16; x++) {
          const float sg = fsigmoid(g[x]), gs = g[x] * sg;   // SiLU(g)
          const float act = gs * u[x];
          // (columns past f: clamped loads, kept out of dw here, out of everything else by what reads it)
          if (c0 + 32 * b + 8 * (x >> 2) + 4 * hi < f) dw = fmaf(h[x], act, dw);
          // d SiLU / dg = sig (1 + g (1 - sig)) = sig + SiLU(g) (1 - sig)
          g[x] = (da[x] * u[x]) * fmaf(gs, 1.f - sg, sg);
          u[x] = da[x] * gs;
          da[x] = act;
        }
        tile_put(t0, l31, hi, 32 * b, g);
        tile_put(t1, l31, hi, 32 * b, u);
        tile_put(t2, l31, hi, 32 * b, da);
        __builtin_amdgcn_sched_barrier(0);   // (interleaved further, the wave runs out of registers)
      }
      dw += __shfl_xor(dw, 32, 64);
      __syncthreads();   // both roles' tiles and the row factors are complete; the sums of the tile before are read
      if (hi == 0) sh.dw[wave][l31] = dw;
    } else {
      __syncthreads();
    }
    // the next tile's operands, the tokens of the one after it, the place of the one after that
    request(col_of(clampi(i + 1) / nt));
    request_rows(expert_of(gid1), tokm);
    take(gid2, row02, rows2);
    tokens(row02, rows2);
    place(i + 3);
    __builtin_amdgcn_sched_barrier(0);
    if (live) {
      {   // per-token sums over the two pairs, bf16 values added in fp32 (expert a's first), rounded once: role A dg, role B du
        const bf16_t *ta = sh.tile[cw][role], *tb = sh.tile[PGB_CW + cw][role];
        bf16_t *out = role ? a.dusum : a.dgsum;
        const bool cvalid = c0 + 8 * cc < f;
#pragma unroll
        for (int p = 0; p < 4; p++) {
          if (8 * p + rr < n && cvalid) {
            const int o = (8 * p + rr) * FT_PITCH + 8 * cc;
            const bf16x8_t va = ld8(ta + o), vb8 = ld8(tb + o);
            bf16x8_t v;
#pragma unroll
            for (int m = 0; m < 8; m++) v[m] = (bf16_t)((float)va[m] + (float)vb8[m]);
            stg8(out, ((uint32_t)sh.tok[8 * p + rr] * (uint32_t)f + c0 + 8 * cc) * 2u, v);
          }
        }
      }
#pragma unroll
      for (int bank = 0; bank < 2; bank++) {
        const bf16_t *t = bank ? t1 : t0;
#pragma unroll
        for (int x = 0; x < 2; x++) {
          f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int ks = 0; ks < 2; ks++)
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ld8(t + (16 * x + l15) * FT_PITCH + 32 * ks + 8 * h4),
                                                          tw[bank][ks], acc, 0, 0, 0);
#pragma unroll
          for (int m = 0; m < 4; m++) sh.T[wave][bank][16 * x + 4 * h4 + m][l15] = acc[m];
        }
      }
#pragma unroll
      for (int q = 0; q < 3; q++) {
        const bf16x8_t pt = ld8_t(&sh.P[role][q][4 * h4 + (l15 >> 2)][4 * (l15 & 3)], 16);
        const bf16_t *t = (q == 0 ? t0 : q == 1 ? t1 : t2) + (4 * h4 + (l15 >> 2)) * FT_PITCH + 4 * (l15 & 3);
#pragma unroll
        for (int j = 0; j < 4; j++)
          dacc[q][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ld8_t(t + 16 * j, FT_PITCH), pt, dacc[q][j], 0, 0, 0);
      }
    }
    if (i + 1 < i1) change(expert_of(gid1), (i + 1) / nt);
    last_rows = n;
    last_cb = cbi;
    gid = gid1, rows = rows1;
    gid1 = gid2, rows1 = rows2;
    __syncthreads();   // the tiles may be overwritten; the wavefronts' rank-r products are complete
  }
  add_waves((i1 - 1) & 1);
  if (e >= 0) flush();
  if (lane == 0)
    for (int b = cb_first; b <= (i1 - 1) / nt; b++) a.masks[(size_t)(wgid + b) * PGB_WAVES + wave] = b == cb_first ? used[0] : used[1];
}

// The three sums from the slots in use, workgroups in ascending order, role A's before role B's; a
// workgroup: one expert, one sum, PGB_COLS columns, a thread all rank entries of one column.
__global__ __launch_bounds__(PGB_COLS) void pg_sums_reduce_kernel(PgBwd a, float scale, float *__restrict__ dB_gate,
                                                             float *__restrict__ dB_up, float *__restrict__ dA_down) {
  const int cb = blockIdx.x, e = blockIdx.y, sum = blockIdx.z, N = a.pc.N, r = a.pc.r, f = a.f;
  const int nt = a.ntiles[0], ncb = gridDim.x, per = pgb_run(nt, ncb, a.nwg);
  const int cw = threadIdx.x >> 6, col = threadIdx.x & 63, c = cb * PGB_COLS + threadIdx.x;
  float acc[16];
#pragma unroll
  for (int q = 0; q < 16; q++) acc[q] = 0.f;
  for (int wg = cb * nt / per; wg <= ((cb + 1) * nt - 1) / per; wg++) {
    for (int role = 0; role < 2; role++) {
      const size_t at = (size_t)(wg + cb) * PGB_WAVES + role * PGB_CW + cw;
      if (!((a.masks[at] >> e) & 1)) continue;
      const float *src = a.slots + ((at * N + e) * 3 + sum) * r * 64 + col;
      float v[16];
#pragma unroll
      for (int q = 0; q < 16; q++) v[q] = src[(q < r ? q : 0) * 64];
#pragma unroll
      for (int q = 0; q < 16; q++) acc[q] += v[q];
    }
  }
  if (c >= f) return;
  if (sum == 2) {
#pragma unroll
    for (int q = 0; q < 16; q++)
      if (q < r) dA_down[((int64_t)e * r + q) * f + c] = scale * acc[q];
    return;
  }
  float *out = (sum ? dB_up : dB_gate) + ((int64_t)e * f + c) * r;
#pragma unroll
  for (int q = 0; q < 16; q += 4)
    if (q < r) *reinterpret_cast<float4 *>(out + q) = make_float4(scale * acc[q], scale * acc[q + 1], scale * acc[q + 2], scale * acc[q + 3]);
}

// The forward has no lower limit on the tokens per pair of experts: the expert-grouped stage would add a
// token's two activations after rounding each to bf16, here they are added in fp32 and rounded once
// (3.3e-3 of the output).
bool fused_pg_ok(const PairCtx &pc, int f) {
  return pc.k == 2 && pc.N <= PG_MAX_EXPERTS && pc.r <= 16 && pc.T > 128 && pc.T <= PG_MAX_TOKENS &&
         f >= 64 && (int64_t)2 * pc.T * f < ((int64_t)1 << 31);
}

// The backward takes at least 24 (rank 8) or 36 (rank 16) tokens per pair of experts that can occur (pairs of
// one adapter's own), or 3400 in all: with fewer, tiles are mostly padding and the expert, with it r columns of
// sums to flush, changes with every tile; the expert-grouped stage, its combine and its sums are ahead then.
// Where those sums are cut into row slices, which costs them another 15 us, 28 are enough at rank 16. Training
// step, us, here / there, rank 16: 7B shape, 8 experts, 784 tokens 675 / 671, 1000 733 / 719, 1050 802 / 801,
// 1300 963 / 972; 12 experts 2000 1236 / 1225, 2400 1558 / 1560; 16 experts 3000 1824 / 1799, 3400 1980 / 1983,
// 4200 2406 / 2409; two adapters of 8, 1900 1275 / 1252, 2048 1274 / 1283; sums cut: 2048 x 5504 784 311 / 332,
// 2048 x 8192 784 385 / 402, 6 experts of the 7B shape 420 446 / 465. Rank 8: 7B shape, 8 experts, 600 532 /
// 530, 784 640 / 643; 16 experts 2200 1516 / 1489, 3000 1742 / 1767. Below 1024 items, column blocks times
// tiles, two workgroups per CU have one each: 1024 x 2752, 1000 tokens 224 / 211, 1500 230 / 235; 512 x 1536,
// 1800 187 / 179, 3000 216 / 218. And few column blocks leave pg_sums_reduce_kernel a long chain of runs: 256 x
// 512, 10000 tokens 288 / 263, 20000 411 / 419; x 704, 7000 252 / 235, 14000 359 / 375; x 1024, 5000 241 / 235,
// 7000 281 / 284.
static bool pg_bwd_size(int f, int T, int N, int Nl, int r) {
  const bool cut = group_outer_mfma_partial_floats(N, r, f, 2 * T, 3) > 0;
  const int64_t blocks = fused_pg_bwd_splits(f), items = blocks * ((T + FT_ROWS - 1) / FT_ROWS);
  const int64_t half_pair = r <= 8 ? 12 : cut ? 14 : 18;
  return (T >= half_pair * N * (Nl - 1) || T >= 3400) && items >= 1024 && items * blocks >= 12000;
}
bool fused_pg_bwd_ok(const PairCtx &pc, int f, int Nl) {
  return fused_pg_ok(pc, f) && pg_bwd_size(f, pc.T, pc.N, Nl, pc.r);
}

int fused_pg_max_tiles(int T, int N) { return (T + FT_ROWS - 1) / FT_ROWS + N * N; }

// Column splits (grid.y).  Measured at the LLaMA shapes: a workgroup pays a few microseconds of
// set-up (metadata chain, first fetches) and of final reduction, so few long workgroups beat many
// short ones, and best of all is a grid that fits the chip in one round (two 4-wave workgroups
// per compute unit: 512 slots).  tiles = T / 32 plus half a ragged tile per pair group.
int fused_pg_splits(int f, int T, int N) {
  const int nblk = (f + FT_SB - 1) / FT_SB;
  const int tiles = (T + FT_ROWS - 1) / FT_ROWS + N * (N - 1) / 4;
  const int fit = 512 / (tiles > 0 ? tiles : 1);
  int s = fit >= 3 ? (fit < 16 ? fit : 16) : 4;
  while (s > 1 && nblk / s < FT_WAVES) s--;
  return s;
}

hipError_t launch_swiglu_fwd_pg(const PairCtx &pc, int f, float s, const int32_t *tok_of_pos,
                                const int32_t *tile_info, const int32_t *ntiles, const void *G,
                                const void *U, const float *Pg_all, const float *Pu_all,
                                const void *B_gate, const void *B_up, const void *A_down,
                                void *a_comb, float *Q_part, float *Q_all, void *Qw,
                                int ldqw, hipStream_t st) {
  if (!fused_pg_ok(pc, f)) return hipErrorInvalidValue;
  const int nsplit = fused_pg_splits(f, pc.T, pc.N);
  const dim3 grid(fused_pg_max_tiles(pc.T, pc.N), nsplit), block(FT_WAVES * 64);
  hipLaunchKernelGGL(swiglu_fwd_pg_kernel, grid, block, 0, st, pc, f, s, tok_of_pos, tile_info, ntiles,
                     (const bf16_t *)G, (const bf16_t *)U, Pg_all, Pu_all, (const bf16_t *)B_gate,
                     (const bf16_t *)B_up, (const bf16_t *)A_down, (bf16_t *)a_comb, Q_part, nsplit);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_reduce_rank_parts(pc, Q_part, nsplit, Q_all, Qw, ldqw, 1, 0, st);
}

int fused_pg_bwd_splits(int f) { return (f + PGB_COLS - 1) / PGB_COLS; }

// Workgroups: two per CU, a tile each at least; never fewer than column blocks, so that a run touches two of
// them at most.
static int pgb_workgroups(int f, int T, int N) {
  const int64_t ncb = fused_pg_bwd_splits(f), tiles = (T + FT_ROWS - 1) / FT_ROWS + N * (N - 1) / 4;
  int64_t n = ncb * tiles;
  n = n > 512 ? 512 : n;
  return (int)(n < ncb ? ncb : n);
}

size_t fused_pg_bwd_floats(int f, int T, int N, int r) {
  const size_t pieces = pgb_workgroups(f, T, N) + fused_pg_bwd_splits(f);
  return pieces * PGB_WAVES * N * 3 * r * 64 + pieces * PGB_WAVES;
}

hipError_t launch_swiglu_bwd_pg(const PairCtx &pc, int f, float s, const int32_t *tok_of_pos,
                                const int32_t *tile_info, const int32_t *ntiles, const void *G,
                                const void *U, const void *H, const float *Pg_all,
                                const float *Pu_all, const float *VB_all, const void *B_gate,
                                const void *B_up, const void *AdT, const void *BgT, const void *BuT,
                                void *dgsum, void *dusum, float *dw_part, float *rank_part, float *slots,
                                float *dB_gate, float *dB_up, float *dA_down, hipStream_t st) {
  if (!fused_pg_ok(pc, f)) return hipErrorInvalidValue;
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e_ = hipFuncSetAttribute(reinterpret_cast<const void *>(swiglu_bwd_pg_kernel),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(PgbShared));
    if (e_ != hipSuccess) return e_;
    attr_set = true;
  }
  const int nwg = pgb_workgroups(f, pc.T, pc.N), ncb = fused_pg_bwd_splits(f);
  const PgBwd a{pc, f, nwg, s, tok_of_pos, tile_info, ntiles, (const bf16_t *)G, (const bf16_t *)U,
                (const bf16_t *)H, Pg_all, Pu_all, VB_all, (const bf16_t *)B_gate, (const bf16_t *)B_up,
                (const bf16_t *)AdT, (const bf16_t *)BgT, (const bf16_t *)BuT, (bf16_t *)dgsum, (bf16_t *)dusum,
                dw_part, rank_part, slots, (uint32_t *)(slots + (size_t)(nwg + ncb) * PGB_WAVES * pc.N * 3 * pc.r * 64)};
  hipLaunchKernelGGL(swiglu_bwd_pg_kernel, dim3(nwg), dim3(PGB_WAVES * 64), sizeof(PgbShared), st, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(pg_sums_reduce_kernel, dim3(ncb, pc.N, 3), dim3(PGB_COLS), 0, st, a, s, dB_gate, dB_up, dA_down);
  return hipGetLastError();
}

}  // namespace mixlora
