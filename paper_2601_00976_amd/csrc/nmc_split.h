// Building blocks of the small-batch kernels: one wavefront per species of a
// pair of points, work-group of NS wavefronts (CDNA4).
#pragma once

#include "nmc_pair.h"

namespace nmc {
namespace splitk {

// What the waves of a work-group contract at points too cold for the rows in
// registers: the nodes' exponent splits and the vectors of every species.
template <int NS>
struct ColdLds {
  SplitExp E[2];             // per point
  double X[NS][4][kLanes];   // per species: the vectors a, b, c, d (see cold_contract)
};

// sum over the species of what their waves left in LDS for point h
template <int NS, int N, int M>
__device__ __forceinline__ void species_sum(const double (&v)[NS][2][M], int h, double (&s)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) s[i] = v[0][h][i];
#pragma unroll
  for (int t = 1; t < NS; ++t)
#pragma unroll
    for (int i = 0; i < N; ++i) s[i] += v[t][h][i];
}

// The four contractions of a species' rates (core_contract, c and d of its
// pair partner) at a point whose grid spans too many powers of two for the
// row: entries regenerated column by column from the splits in LDS, in a rolled
// loop that needs few registers (such points are rare, and rows held for them
// would cost the others a wave per SIMD).  CORE: every entry is
// b^2 = exp(-|e_q - e_j| / T) and the factors are on the vectors; otherwise
// the four kernels' entries without their factor A e_q e_j, every one at most
// 1 (u = 2^(x_q - x_j) and v = 2^(x_j - x_q): the one not above 1 is b, the
// other its reciprocal or +inf; Phi_in = min(u, v^3), Phi_out = min(u^3, v),
// Phi_ann = min(u^2, v^2) and Phi_pro = G of the higher node).  The work-group
// calls it together; a, b, c, d are this wave's own vectors.
template <int NS, bool CORE>
__device__ __forceinline__ void cold_contract(ColdLds<NS>& S, int sp, int pa, int h, int q, double a, double b,
                                              double c, double d, double& eN, double& oN, double& aP, double& eP) {
  const int lane = 32 * h + q;
  S.X[sp][0][lane] = a;
  S.X[sp][1][lane] = b;
  S.X[sp][2][lane] = c;
  S.X[sp][3][lane] = d;
  __syncthreads();
  const SplitExp& E = S.E[h];
  const double Pq = E.P2[q], Rq = E.R2[q], Gq = E.G[q];
  const int nq = E.n2[q];
  eN = oN = aP = eP = 0.0;
#pragma unroll 1
  for (int j = 0; j < 32; ++j) {
    const int e = nq - E.n2[j];
    const double u = ldexp(Pq * E.R2[j], e), v = ldexp(E.P2[j] * Rq, -e);
    const double u2 = u * u, v2 = v * v, fa = min_f64(u2, v2);
    const double fi = CORE ? fa : min_f64(u, v2 * v), fo = CORE ? fa : min_f64(u2 * u, v);
    const double fp = CORE ? fa : min_f64(E.G[j], Gq);
    const int l = 32 * h + j;
    eN = __builtin_fma(fi, S.X[sp][0][l], eN);
    oN = __builtin_fma(fo, S.X[sp][1][l], oN);
    aP = __builtin_fma(fa, S.X[pa][2][l], aP);
    eP = __builtin_fma(fp, S.X[pa][3][l], eP);
  }
  __syncthreads();
}

// the point's splits at its current temperature (every wave writes the same)
template <int NS>
__device__ __forceinline__ void cold_splits(ColdLds<NS>& S, int h, int q, const ExpSplit& xs) {
  SplitExp& E = S.E[h];
  E.P2[q] = xs.P;
  E.R2[q] = xs.R;
  E.n2[q] = xs.n;
  const double R2 = xs.R * xs.R;
  E.G[q] = ldexp(R2 * R2, -4 * xs.n);  // exp(-2 e / T)
  __syncthreads();
}

}  // namespace splitk
}  // namespace nmc
