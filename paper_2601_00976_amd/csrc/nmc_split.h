// Building blocks of the small-batch kernels: one wavefront per species of a
// pair of points, work-group of NS wavefronts (CDNA4).
#pragma once

#include "nmc_pair.h"

namespace nmc {
namespace splitk {

// Sums over the half-wave of the inner convergence test for the one species of
// a wave, by the tree of spread_conv_sums (mirrored lanes add the same pairs):
// the squared changes of its moments, two or four of them, spread over the
// lanes (every lane has one), and the squared new D in every lane.
__device__ __forceinline__ double conv_tail(double x) {
  x += dpp<0x141>(x);  // row_half_mirror
  x += dpp<0xB1>(x);   // quad_perm [1,0,3,2]
  x += dpp<0x4E>(x);   // quad_perm [2,3,0,1]
  return x;
}
__device__ __forceinline__ void conv_sums(const double (&d)[2], double xn, double& y, double& n) {
  const double a = halve16(d[0], d[1]), b = halve16(xn, xn);
  y = conv_tail(a + dpp<0x140>(a));  // row_mirror
  n = conv_tail(b + dpp<0x140>(b));
}
__device__ __forceinline__ void conv_sums(const double (&d)[4], double xn, double& y, double& n) {
  const double b = halve16(xn, xn);
  y = conv_tail(fold_pair<0x140, 0x3>(halve16(d[0], d[2]), halve16(d[1], d[3])));
  n = conv_tail(b + dpp<0x140>(b));
}

// any lane of half h of this wave
__device__ __forceinline__ bool half_any(bool b, int h) {
  const uint64_t m = __builtin_amdgcn_ballot_w64(b);
  return (h ? m >> 32 : m & 0xffffffffull) != 0;
}

// The lane's pair factors at a point whose grid spans too many powers of two
// for scaled factors (direct_row_regs), from the point's exponent splits in
// LDS: of the two orientations 2^(x_q - x_j) and 2^(x_j - x_q) the smaller is
// b = exp(-|e_q - e_j| / (2T)).  CORE: b^2; otherwise signed as in
// signed_contract (+b where j is the upper node); the values of
// pair_tile_rows, the diagonal written as its callers do.  The work-group calls
// it together, every wave with the same values.  2048 points of 0.13-0.2 MeV took
// 128 us so, 435 us with every column regenerated in every inner iteration, in
// the signed form; the symmetric one, up to kSymBits, takes 4% less.
template <bool CORE>
__device__ __forceinline__ void cold_rows(SplitExp& E, int q, const ExpSplit& xs, double (&B)[16], double& k) {
  E.P2[q] = xs.P;
  E.R2[q] = xs.R;
  E.n2[q] = xs.n;
  __syncthreads();
  auto entry = [&](int j) {
    const int e = xs.n - E.n2[j];
    const double b = min_f64(ldexp(xs.P * E.R2[j], e), ldexp(E.P2[j] * xs.R, -e));
    return CORE ? (j == q ? 1.0 : b * b) : (j > q ? b : j == q ? -1.0 : -b);
  };
  const int r16 = q & 16;
#pragma unroll
  for (int j = 0; j < 16; ++j) B[j] = entry(r16 + j);
  k = entry(r16 ? 15 : 16);
  __syncthreads();
}

// One column of signed_split (lane L of the 16-lane row).
template <int L>
__device__ __forceinline__ void signed_column(double& eN, double& oN, double& aP, double& eP, double x, double y,
                                              double xp, double hyp, double fi, double fo, double fa) {
  asm volatile(
      "s_nop 1\n"
      "v_fmac_f64_dpp %0, %4, %8 row_newbcast:%11 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %5, %9 row_newbcast:%11 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %2, %6, %10 row_newbcast:%11 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %3, %7, %10 row_newbcast:%11 row_mask:0xf bank_mask:0xf\n"
      : "+v"(eN), "+v"(oN), "+v"(aP), "+v"(eP)
      : "v"(x), "v"(y), "v"(xp), "v"(hyp), "v"(fi), "v"(fo), "v"(fa), "i"(L));
}

// signed_contract with the pair partner's vectors apart: eN = Phi_in x,
// oN = Phi_out y, aP = Phi_ann xp, eP = Phi_ann hyp
__device__ __forceinline__ void signed_split(const double (&B)[16], double k, double x, double y, double xp, double hyp,
                                             double& eN, double& oN, double& aP, double& eP) {
  eN = oN = aP = eP = 0.0;
  static_for<0, 16>([&](auto jj) __attribute__((always_inline)) {
    constexpr int j = decltype(jj)::value;
    double sb = B[j];
    asm volatile("" : "+v"(sb));  // the products are not shared between calls (48 more registers)
    const double b2 = sb * sb, c3 = sb * b2;
    signed_column<j>(eN, oN, aP, eP, x, y, xp, hyp, pairk::max_neg_f64(sb, c3), pairk::max_neg_f64(c3, sb), b2);
  });
  const double k2 = k * k, k3 = k * k2, kN = pairk::max_neg_f64(k, k3), kO = pairk::max_neg_f64(k3, k);
  const double z0 = mirror32(eN), z1 = mirror32(oN), z2 = mirror32(aP), z3 = mirror32(eP);
  pairk::cross_fmac(eN, oN, aP, eP, z0, z1, z2, z3, kN, kO, k2, k2);
}

}  // namespace splitk
}  // namespace nmc
