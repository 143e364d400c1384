// Per-token pieces that run in launches of their own (csrc/elementwise.hip) and beside others
// (csrc/tail.hip).
#pragma once
#include "common.h"

namespace mixlora {

// ---- out[t, :] = sum_j (w[t,j] or 1) * in_grp[row_of_pair[t,j], :] ------------------------------
// Gather form of the weighted combine (Eq. 6; Algorithm 1 line 15): each output row is written
// once, by one thread per 8 columns, slots added in ascending order (deterministic).
template <typename E>
__device__ __forceinline__ void pair_combine_body(const PairCtx &pc, int width,
                                                  const E *__restrict__ in_grp,
                                                  E *__restrict__ out, int weighted, int t, int by) {
  // a thread owns two 8-column chunks, 2048 columns apart: 2k independent loads in flight
  const int c0 = (by * 512 + threadIdx.x) * 8;
  const int c1 = c0 + 2048;
  if (c0 >= width) return;
  const bool two = c1 < width;
  float acc0[8] = {0, 0, 0, 0, 0, 0, 0, 0}, acc1[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int j = 0; j < pc.k; j++) {
    const int p = t * pc.k + j;
    const float w = weighted ? pc.w[p] : 1.f;
    const E *src = in_grp + (int64_t)pc.row_of_pair[p] * width;
    Vec8<E> v0, v1;
    v0.load(src + c0);
    if (two) v1.load(src + c1);
#pragma unroll
    for (int i = 0; i < 8; i++) acc0[i] = fmaf(w, v0.get(i), acc0[i]);
    if (two) {
#pragma unroll
      for (int i = 0; i < 8; i++) acc1[i] = fmaf(w, v1.get(i), acc1[i]);
    }
  }
  Vec8<E> o;
#pragma unroll
  for (int i = 0; i < 8; i++) o.set(i, acc0[i]);
  o.store(out + (int64_t)t * width + c0);
  if (two) {
#pragma unroll
    for (int i = 0; i < 8; i++) o.set(i, acc1[i]);
    o.store(out + (int64_t)t * width + c1);
  }
}

inline int pair_combine_slices(int width) { return (width + 4095) / 4096; }   // workgroups per token

}  // namespace mixlora
