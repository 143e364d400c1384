// Routing of one token by one lane, for the launches that route many tokens per workgroup.
#pragma once
#include "common.h"

namespace mixlora {

// Softmax, top-k and renormalisation of one token by one lane, with the operations and their order of
// route_token (csrc/router.hip), of which this is the serial form: sums over experts as a butterfly
// would take them, ties to the lower index, kept experts closed, NaN ranked with -inf.
// PROBS: p[] gets all probabilities; without, only the kept ones are divided out.
template <int NMAX, bool PROBS>
__device__ __forceinline__ void route_lane(float (&z)[NMAX], int lo, int Nl, int k, float (&p)[NMAX],
                                           int (&es)[ROUTE_MAX_K], float (&ws)[ROUTE_MAX_K]) {
  float sum[NMAX];
  float zmax = -INFINITY;
#pragma unroll
  for (int n = 0; n < NMAX; n++) {
    if (n < lo || n >= lo + Nl) z[n] = -INFINITY;
    zmax = fmaxf(zmax, z[n]);
  }
#pragma unroll
  for (int n = 0; n < NMAX; n++) p[n] = sum[n] = n >= lo && n < lo + Nl ? expf(z[n] - zmax) : 0.f;
#pragma unroll
  for (int o = NMAX / 2; o > 0; o >>= 1)
#pragma unroll
    for (int n = 0; n < o; n++) sum[n] += sum[n + o];
  unsigned open = 0;
#pragma unroll
  for (int n = 0; n < NMAX; n++) {
    if constexpr (PROBS) p[n] /= sum[0];
    if (!(z[n] == z[n])) z[n] = -INFINITY;
    if (n >= lo && n < lo + Nl) open |= 1u << n;
  }
  float ksum = 0.f;
#pragma unroll
  for (int j = 0; j < ROUTE_MAX_K; j++) {
    es[j] = 0;
    ws[j] = 0.f;
    if (j < k) {
      float m = -INFINITY;
#pragma unroll
      for (int n = 0; n < NMAX; n++)
        if ((open >> n) & 1) m = fmaxf(m, z[n]);
      int e = -1;
      float pe = 0.f;
#pragma unroll
      for (int n = NMAX - 1; n >= 0; n--)
        if (((open >> n) & 1) && z[n] == m) {
          e = n;
          pe = p[n];
        }
      if constexpr (!PROBS) pe /= sum[0];
      open &= ~(1u << e);
      ksum += pe;
      es[j] = e;
      ws[j] = pe;
    }
  }
#pragma unroll
  for (int j = 0; j < ROUTE_MAX_K; j++) ws[j] /= ksum;
}

}  // namespace mixlora
