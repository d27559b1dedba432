// Adjoint (implicit-function-theorem) kernels of the coupling solve on CDNA4.
//
// At the converged state x = (D, Ye, e) of a point the reduced residual
//   R_D = D (1 + dtau chi) - D* - dtau eta          (Eq. implicitMomentsNodal, v = 0)
//   R_Y = Ye - Ye* + K sum_s g_s sum_q W_q (D - D*)  (Eq. implicitFluidNodal)
//   R_e = e  - e*  + K sum_s d_s sum_q W3_q (D - D*)
// vanishes (the flux moments drop out: nothing depends on I when v = 0).
// With J = dR/dx = [[A, B], [C, 1]] (A: moment block, B: the Ye / e columns
// through T(e, Ye) and mu(Ye, T), C: the conservation rows) the transposed
// system J^T lambda = dL/dx is solved by a Schur complement on the two matter
// unknowns:
//   Z = A^-T C^T,  (1 - B^T Z) lambda_m = (gY, -gE),  lambda_D = -Z lambda_m,
// and dL/dtheta_j = -lambda_D^T dR_D/dtheta_j for theta = (s_1..s_nq, a_nes,
// a_pair), L = gE (e* - e) + gY (Ye - Ye*).
//
// Two ways to solve for Z, both FP64:
//
// Iteration (the usual one, PairAdjoint): two points per wavefront as in the
// forward kernel.  A^T = G - N with G its diagonal is iterated as
// z <- G^-1 (c + N z).  The W-scaled columns of A are strictly diagonally
// dominant, so this always converges, and over a time step of a transport
// code N is small against G: on the radial profile at dtau = 1e-3 km it takes
// 3.7 iterations on average and 11 at most to reach rounding, each one the
// forward solve's contraction on the symmetric core (24 n^2 multiply-adds for
// both columns of C) where an elimination takes (2/3) (64^3 + 32^3).
//
// A long step or strong coupling makes N large: the changes then have to keep a
// pace (kAdjPace bits per iteration, looked at after 2, 6 and 12), and a point
// that falls behind is left to the elimination at once.
//
// Elimination (PointAdjoint): for points that the iteration does not settle
// (slow convergence, a non-finite value) or whose grid spans too many powers
// of two for it, in a second kernel with a work-group per point.  A is block
// diagonal over pair-coupled species: NES couples the nodes of one species,
// pair processes couple a species with its partner, so with species in id
// order the blocks are (nu_e, anti-nu_e) of size 64 and nu_x of size 32.  Each
// block is factorised in registers, one wavefront per
// point: lane r holds row r of A^T (column r of A) and the two right-hand
// sides.  Block Gauss-Jordan elimination with 2 x 2 pivot blocks runs without
// row exchanges, broadcasting the two pivot rows of each step through LDS.
//
// Every work-group adds its points' terms in order and writes one row of
// partial sums (one of the elimination only if it had a point); a last kernel
// adds the rows of each column in a fixed order.
//
// us of a call, eliminating every point / without the pace and two points of a
// pair eliminated one after the other / so: 8 points at 0.5 km, none settling,
// 70 / 117 / 54; 65536 such points 1954 / 2831 / 2086; the whole profile at 0.5
// km, 65536 points, 1946 / 959 / 829; 65536 points of 0.1-0.2 MeV 1946 / 2063 /
// 1910; at 1e-3 km, all settling, 1951 / 305 / 303.  Where the caller asks for
// them, the per-point terms go to a (P, nq + 2) array as well.
#include "nmc_pair.h"

namespace nmc {
namespace {

constexpr int NQ = 32;

template <int NS>
struct AdjLds {
  ModelLds m;
  SplitExp E;
  double tb[32 * kTileStride];  // pair factors b = exp(-|e_q - e_p| / (2T)) of the kernels
  double D[NS][NQ];
  // per-row results, row = (species, node)
  double chi[NS][NQ];         // total opacity chi of the row
  double b0[NS][NQ], b1[NS][NQ];  // dR_D / dYe, dR_D / de
  double da[NS][NQ], dp[NS][NQ], ds[NS][NQ];  // dR_D / d a_nes, / d a_pair, / d s_q
  double z0[NS][NQ], z1[NS][NQ];  // Z = A^-T C^T
  alignas(16) double prow[2 * (2 * NQ + 2)];  // pivot-row buffers of the block factorisation
};

// ds_write2_b64 of (a, b) to LDS bytes base + 8 J and base + 8 (J + 1)
template <int J>
__device__ __forceinline__ void lds_write2_f64(uint32_t base, double a, double b) {
  static_assert(J + 1 <= 255, "ds_write2_b64 offsets are 8-bit");
  asm volatile("ds_write2_b64 %0, %1, %2 offset0:%3 offset1:%4" : : "v"(base), "v"(a), "v"(b), "i"(J), "i"(J + 1)
               : "memory");
}

// R[J + i] += bcast_{L + i}(u) b + bcast_{L + i}(w) a for i = 0..3, the
// column values u, w taken from lane L + i of the lane's 16-lane row
// (v_fmac_f64_dpp row_newbcast): the b term first, then the a term, each one
// rounding.  The leading s_nop covers a VALU write of u or w just before.
template <int L>
__device__ __forceinline__ void elim_cols4(double& r0, double& r1, double& r2, double& r3, double u, double w,
                                           double a, double b) {
  asm volatile(
      "s_nop 1\n"
      "v_fmac_f64_dpp %0, %5, %7 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %5, %7 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %2, %5, %7 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %3, %5, %7 row_newbcast:%11 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %0, %4, %6 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %1, %4, %6 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %2, %4, %6 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f64_dpp %3, %4, %6 row_newbcast:%11 row_mask:0xf bank_mask:0xf\n"
      : "+v"(r0), "+v"(r1), "+v"(r2), "+v"(r3)
      : "v"(u), "v"(w), "v"(a), "v"(b), "i"(L), "i"(L + 1), "i"(L + 2), "i"(L + 3));
}

// Solves A^T z = c for one diagonal block of size N (lanes 0..N-1 active):
// lane r enters with R = row r of A^T and c = (c0, c1) its right-hand sides
// and leaves with (z0, z1) = entry r of the two solutions.  Returns false if
// a pivot block was singular or non-finite, detected as a non-finite
// solution entry (such a block turns the multipliers or the final quotients
// into inf or NaN, which propagate into z).
//
// Block Gauss-Jordan elimination with 2 x 2 pivot blocks and no row
// exchanges: with D in [0, 1] and non-negative kernels, diag(W) A is strictly
// diagonally dominant by columns (the off-diagonal column sums of the
// W-scaled NES and pair terms equal the kernel part of the diagonal opacity,
// leaving a margin W_p (1 + dtau chi^EmAb_p)), so A^T with its columns scaled
// by W is dominant by rows; elimination without pivoting, Gauss-Jordan
// included, is stable for such matrices, and their diagonal blocks and Schur
// complements stay dominant, so every 2 x 2 pivot block is nonsingular.
// Step k (even) removes columns k and k+1 from every row but k and k+1 (lanes
// k and k+1) with the multipliers [R[k], R[k+1]] B^-1 of the pivot block B.
// The two lanes write their rows (from column k on) and right-hand sides to
// two LDS row buffers; every lane then loads, per group of 16 columns, one
// entry of each pivot row (lane L of a 16-lane row loads column 16 g + L), and
// the update FMAs take column 16 g + L from lane L of the lane's row by DPP
// broadcast.  All lanes run the FMAs (a DPP source lane must be active); the
// pivot rows have zero multipliers, so their entries are unchanged.  The
// update starts at the 4-column block of column k + 2; the columns of that
// block left of k + 2 are updated too: they are eliminated columns or the
// row's own pivot block, which the row keeps in registers when it is
// eliminated, and are never read again.  Rows above the pivot are
// updated by the same instructions as the rows below, so the elimination
// costs no more than a one-sided one, and at the end every pivot pair holds
// only its own block: z = B^-1 c for each pair, from the partner's
// right-hand sides by DPP, with no back substitution.  A single wavefront
// runs the work-group, so its LDS accesses complete in program order and no
// barrier is needed.
template <int N>
__device__ __forceinline__ bool solve_block_transposed(double (&R)[N], double c0, double c1, double& z0,
                                                       double& z1, double* prow_generic) {
  static_assert(N % 16 == 0, "2 x 2 pivot blocks, 16-column groups");
  typedef double f64x2 __attribute__((ext_vector_type(2)));
  typedef __attribute__((address_space(3))) double lds_f64;
  typedef __attribute__((address_space(3))) f64x2 lds_f64x2;
  constexpr int RS = N + 2;  // doubles per row buffer: entries 0..N-1, right-hand sides at N, N+1
  const int lane = opaque((int)threadIdx.x);
  const int col = lane & 15;
  // the lane's pivot block, kept when its pair is eliminated: lane k (even)
  // solves z_k = (a11 c_k - a01 c_k+1) / det, lane k+1 z_k+1 = (a00 c_k+1 -
  // a10 c_k) / det, so each keeps its (x, y) = (a11, a01) or (a00, a10)
  double bx = 0.0, by = 0.0, brd = 0.0;
  static_for<0, N / 2>([&](auto kk) __attribute__((always_inline)) {
    constexpr int k = 2 * decltype(kk)::value;
    lds_f64* prow = (lds_f64*)prow_generic;
    lds_f64x2* prow2 = (lds_f64x2*)prow;
    // the pivot block B = [[a00, a01], [a10, a11]] (rows k, k+1, columns k, k+1)
    const double a00 = readlane(R[k], k), a01 = readlane(R[k + 1], k);
    const double a10 = readlane(R[k], k + 1), a11 = readlane(R[k + 1], k + 1);
    if (lane == k || lane == k + 1) {
      // rows k and k+1 (columns k..N-1) to their buffers: ds_write2_b64 from
      // one base register per lane with 8-byte-unit offsets
      const uint32_t base = (uint32_t)(uintptr_t)prow + (uint32_t)((lane - k) * RS * 8);
      static_for<0, (N - k) / 2>([&](auto ii) __attribute__((always_inline)) {
        constexpr int j = k + 2 * decltype(ii)::value;
        lds_write2_f64<j>(base, R[j], R[j + 1]);
      });
      lds_write2_f64<N>(base, c0, c1);
    }
    const double rdet = rcp_nr(a00 * a11 - a01 * a10);
    if (lane == k) {
      bx = a11;
      by = a01;
      brd = rdet;
    }
    if (lane == k + 1) {
      bx = a00;
      by = a10;
      brd = rdet;
    }
    const bool other = lane != k && lane != k + 1;
    const double nl0 = other ? -((R[k] * a11 - R[k + 1] * a10) * rdet) : 0.0;
    const double nl1 = other ? -((R[k + 1] * a00 - R[k] * a01) * rdet) : 0.0;
    static_for<(k + 2) / 16, N / 16>([&](auto gg) __attribute__((always_inline)) {
      constexpr int g = decltype(gg)::value;
      const double u = prow[16 * g + col], w = prow[RS + 16 * g + col];
      // in the group of column k + 2, the 4-column blocks left of it hold
      // only dead entries (eliminated columns, or the pivot blocks kept in
      // registers): skipped
      constexpr int q0 = g == (k + 2) / 16 ? ((k + 2) % 16) / 4 : 0;
      static_for<q0, 4>([&](auto qq) __attribute__((always_inline)) {
        constexpr int j = 16 * g + 4 * decltype(qq)::value;
        elim_cols4<j % 16>(R[j], R[j + 1], R[j + 2], R[j + 3], u, w, nl0, nl1);
      });
    });
    const f64x2 cu = prow2[N / 2], cv = prow2[(RS + N) / 2];
    c0 = __builtin_fma(nl0, cu.x, __builtin_fma(nl1, cv.x, c0));
    c1 = __builtin_fma(nl0, cu.y, __builtin_fma(nl1, cv.y, c1));
  });
  // each pivot pair (k, k+1) now solves its own block; the partner lane is
  // lane ^ 1 (quad_perm [1,0,3,2])
  const double o0 = dpp<0xB1>(c0), o1 = dpp<0xB1>(c1);
  z0 = (bx * c0 - by * o0) * brd;
  z1 = (bx * c1 - by * o1) * brd;
  // a singular or non-finite pivot block makes some entry of the solution
  // non-finite
  return __builtin_amdgcn_ballot_w64(lane < N && !(isfinite(z0) && isfinite(z1))) == 0;
}

template <int NS>
struct PointAdjoint {
  // Rows of A^T of one block of species [S0, S0 + NB): lane r = 32 si + p
  // holds column (S0 + si, p) of A.  Entries (Jacobian of R_D):
  //   same species (NES):  -dtau W_p [(1 - D_q) Phi_in[q][p] + D_q Phi_out[q][p]]
  //   partner species:     +dtau W_p [D_q Phi_ann[q][p] + (1 - D_q) Phi_pro[q][p]]
  //   diagonal:            1 + dtau chi_(s, p)
  // with the kernels at the point's amplitudes; Phi_out[q][p] = Phi_in[p][q].
  // The kernels are formed from the pair factors b: with c = rho e_q e_p,
  // Phi_in[q][p] = c (p > q ? b : b^3), Phi_out[q][p] = c (q > p ? b : b^3),
  // Phi_ann = c b^2, Phi_pro = c G_max(q, p).
  template <int S0, int NB>
  __device__ __forceinline__ static void block_rows(AdjLds<NS>& S, double dtau, double rho, double a_nes,
                                                    double a_pair, double (&R)[32 * NB]) {
    constexpr int ST = kTileStride;
    const int lane = opaque((int)threadIdx.x);  // laundered: lane-derived indices are not hoisted out of the point loop
    const int h = lane >> 5, p = lane & 31;
    const int si = NB == 2 ? h : 0;
    const int sp = S0 + si;  // species of this lane's column
    const double rwe = rho * S.m.w2[p] * S.m.eps[p];
    const double dwn = dtau * a_nes * rwe, dwp = dtau * a_pair * rwe;
    const double diag = 1.0 + dtau * S.chi[sp][p];
    const double Gp = S.E.G[p];
    // the moments are re-read here (an opaque zero offset keeps the compiler
    // from carrying the values loaded for the contractions through the
    // factorisation of the previous block in registers)
    int z = 0;
    asm volatile("" : "+s"(z));
    const double* __restrict__ Db = &S.D[S0][z];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const double eq = S.m.eps[q], Gq = S.E.G[q];
      const double b = S.tb[q * ST + p], b2 = b * b, b3 = b2 * b;
      const double fin = p > q ? b : b3, fout = q > p ? b : b3;
      const double fpro = fmin(Gq, Gp);  // G of the higher node: G falls with energy
      const double nq = -dwn * eq, pq = dwp * eq;
      // row (s, q), column (sp, p): NES if s = sp, pair if s is sp's partner
      auto nes = [&](double d) { return nq * __builtin_fma(d, fout - fin, fin); };
      auto pair = [&](double d) { return pq * __builtin_fma(d, b2 - fpro, fpro); };
      const double dg = q == p ? diag : 0.0;
      if constexpr (NB == 2) {
        // d is the moment of the row's species: the lane's own species for
        // its NES row, the partner's for its pair row
        const double d0 = Db[q], d1 = Db[NQ + q];
        const double vn = nes(si == 0 ? d0 : d1) + dg, vp = pair(si == 0 ? d1 : d0);
        R[q] = si == 0 ? vn : vp;
        R[32 + q] = si == 0 ? vp : vn;
      } else {
        const double d = Db[q];
        R[q] = nes(d) + pair(d) + dg;
      }
      if ((q & 3) == 3) asm volatile("" ::: "memory");
    }
  }

  template <int S0, int NB>
  __device__ __forceinline__ static bool block_solve(AdjLds<NS>& S, const DevModel* md, double dtau, double rho,
                                                     double a_nes, double a_pair, double K) {
    double R[32 * NB];
    block_rows<S0, NB>(S, dtau, rho, a_nes, a_pair, R);
    const int lane = opaque((int)threadIdx.x);  // laundered: lane-derived indices are not hoisted out of the point loop
    const int h = lane >> 5, p = lane & 31;
    const int sp = S0 + (NB == 2 ? h : 0);
    // right-hand sides: column (sp, p) of the conservation rows C
    const double c0 = K * md->ig[sp] * S.m.w2[p];
    const double c1 = K * md->imult[sp] * S.m.w3[p];
    double z0, z1;
    const bool ok = solve_block_transposed<32 * NB>(R, c0, c1, z0, z1, S.prow);
    if (lane < 32 * NB) {
      S.z0[sp][p] = z0;
      S.z1[sp][p] = z1;
    }
    __syncthreads();
    return ok;
  }

  // the terms of a point that has any: its s_q term in lane q (lanes 0..31), its a_nes
  // and a_pair terms in every lane
  __device__ static void run(const AdjArgs& a, int64_t pt, AdjLds<NS>& S, double& g_s, double& g_nes,
                             double& g_pair) {
    constexpr int ST = kTileStride;
    const DevModel* __restrict__ md = a.mdl;
    const int lane = opaque((int)threadIdx.x);  // laundered: lane-derived indices are not hoisted out of the point loop
    const int h = lane >> 5, q = lane & 31;
    const int64_t base = pt * (int64_t)(NS * NQ);
    if (lane < 32) {
#pragma unroll
      for (int t = 0; t < NS; ++t) S.D[t][lane] = a.D[base + md->ext[t] * NQ + lane];
    }
    const double rho = a.rho11[pt], ye = a.ye[pt], e = a.e[pt];
    const double chi0 = a.chi0 ? a.chi0[pt] : md->chi_ref * rho;
    const double dtau = a.dtau;
    // EOS and its derivatives
    const double r3 = cbrt(rho);
    const double ia = 1.0 / (md->eos_a * (1.0 + ye));
    const double T = (e - md->eos_b * ye43(ye) * r3) * ia;
    const double mu = md->mu_a * (ye - md->mu_ye0) * r3 + md->mu_b * log(T / md->mu_t0);
    const double invT = 1.0 / T;
    const double dT_de = ia;
    const double dT_dye = -(4.0 / 3.0) * md->eos_b * cbrt(ye) * r3 * ia - T / (1.0 + ye);
    const double dmu_dye = md->mu_a * r3 + md->mu_b * invT * dT_dye;
    const double dmu_de = md->mu_b * invT * dT_de;
    const double K = md->kcoup / rho;
    const unsigned flags = md->flags;
    const double a_nes = (flags & NMC_NES) ? S.m.theta[NQ] : 0.0;
    const double a_pair = (flags & NMC_PAIR) ? S.m.theta[NQ + 1] : 0.0;
    split_exp_prepare(S.m, invT, S.E);

    // ---- per-row contractions with unit-amplitude kernels (A = rho11) ----
    // group 0: species h (ns >= 2) or 0 (ns = 1, lanes < 32); group 1: nu_x (ns = 3, lanes < 32)
    constexpr int NG = NS == 3 ? 2 : 1;
    int sg[NG], sbg[NG];
    bool on[NG];
    sg[0] = NS >= 2 ? h : 0;
    on[0] = NS >= 2 || lane < 32;
    if constexpr (NG == 2) {
      sg[1] = 2;
      on[1] = lane < 32;
    }
#pragma unroll
    for (int g = 0; g < NG; ++g) sbg[g] = NS == 3 ? (sg[g] < 2 ? 1 - sg[g] : 2) : (NS == 2 ? 1 - sg[g] : 0);
    const double eq = S.m.eps[q];
    // en, on (NES in / out), an, ep (pair ann / pro) and their temperature
    // derivatives times T^2
    double en[NG], onn[NG], an[NG], ep[NG], dn[NG], dout[NG], dan[NG], dpr[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) en[g] = onn[g] = an[g] = ep[g] = dn[g] = dout[g] = dan[g] = dpr[g] = 0.0;
    fill_tile<kTilePairFactor>(S.m, S.E, 1.0, h, q, S.tb);
    __syncthreads();
    // the kernels without their common factor rho e_q (applied to the sums)
    const double Gq = S.E.G[q];
#pragma unroll 2
    for (int p = 0; p < NQ; ++p) {
      const double epp = S.m.eps[p], we = S.m.w2[p] * epp, dl = eq - epp, adl = fabs(dl);
      const double b = S.tb[q * ST + p], b2 = b * b, b3 = b2 * b;
      const bool up = p > q;
      const double tin = we * (up ? b : b3), tout = we * (up ? b3 : b);
      const double tann = we * b2, tpro = we * fmin(S.E.G[p], Gq);
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        const double d = S.D[sg[g]][p], db = S.D[sbg[g]][p];
        en[g] = __builtin_fma(tin, d, en[g]);
        dn[g] = __builtin_fma(tin * (adl + 0.5 * dl), d, dn[g]);
        onn[g] = __builtin_fma(tout, 1.0 - d, onn[g]);
        dout[g] = __builtin_fma(tout * (adl - 0.5 * dl), 1.0 - d, dout[g]);
        an[g] = __builtin_fma(tann, db, an[g]);
        dan[g] = __builtin_fma(tann * adl, db, dan[g]);
        ep[g] = __builtin_fma(tpro, 1.0 - db, ep[g]);
        dpr[g] = __builtin_fma(tpro * (adl + eq + epp), 1.0 - db, dpr[g]);
      }
    }
    {
      const double sc = rho * eq;
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        en[g] *= sc;
        dn[g] *= sc;
        onn[g] *= sc;
        dout[g] *= sc;
        an[g] *= sc;
        dan[g] *= sc;
        ep[g] *= sc;
        dpr[g] *= sc;
      }
    }
    // ---- per-row Jacobian pieces ----------------------------------------
    {
      const double shape = chi0 * S.m.shape[q];
      const double iT2 = invT * invT;
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        if (!on[g]) continue;
        const int s = sg[g];
        const double chia = (flags & NMC_EMAB) ? md->iemab[s] * S.m.theta[q] * shape : 0.0;
        const double x = (eq - md->imusign[s] * mu) * invT;
        const double ex = exp(-fabs(x));
        const double r = 1.0 / (1.0 + ex);
        const double f = x > 0.0 ? ex * r : r;   // Fermi-Dirac D_eq
        const double fc = x > 0.0 ? r : ex * r;  // 1 - D_eq
        const double ddeq_dT = f * fc * x * invT;
        const double ddeq_dmu = f * fc * md->imusign[s] * invT;
        const double Dq = S.D[s][q];
        const double chi = chia + a_nes * (en[g] + onn[g]) + a_pair * (ep[g] + an[g]);
        const double deta_dT = chia * ddeq_dT + (a_nes * dn[g] + a_pair * dpr[g]) * iT2;
        const double dchi_dT = (a_nes * (dn[g] + dout[g]) + a_pair * (dpr[g] + dan[g])) * iT2;
        const double dR_dT = dtau * (Dq * dchi_dT - deta_dT);
        const double dR_dmu = -dtau * chia * ddeq_dmu;
        S.chi[s][q] = chi;
        S.b0[s][q] = dR_dT * dT_dye + dR_dmu * dmu_dye;
        S.b1[s][q] = dR_dT * dT_de + dR_dmu * dmu_de;
        S.da[s][q] = (flags & NMC_NES) ? dtau * (Dq * (en[g] + onn[g]) - en[g]) : 0.0;
        S.dp[s][q] = (flags & NMC_PAIR) ? dtau * (Dq * (ep[g] + an[g]) - ep[g]) : 0.0;
        S.ds[s][q] = (flags & NMC_EMAB) ? dtau * shape * md->iemab[s] * (Dq - f) : 0.0;
      }
    }
    __syncthreads();

    // ---- Z = A^-T C^T, block by block ------------------------------------
    // (kernels at unit amplitude a = 1, i.e. A = rho11, scaled by a_nes, a_pair)
    bool ok;
    if constexpr (NS == 1) {
      ok = block_solve<0, 1>(S, md, dtau, rho, a_nes, a_pair, K);
    } else {
      ok = block_solve<0, 2>(S, md, dtau, rho, a_nes, a_pair, K);
      if constexpr (NS == 3) ok = block_solve<2, 1>(S, md, dtau, rho, a_nes, a_pair, K) && ok;
    }

    // ---- Schur complement on (Ye, e), multipliers and gradient ------------
    double v4[4] = {0.0, 0.0, 0.0, 0.0};
    if (lane < 32) {
#pragma unroll
      for (int t = 0; t < NS; ++t) {
        v4[0] += S.b0[t][q] * S.z0[t][q];
        v4[1] += S.b0[t][q] * S.z1[t][q];
        v4[2] += S.b1[t][q] * S.z0[t][q];
        v4[3] += S.b1[t][q] * S.z1[t][q];
      }
    }
    double bz[4];
    wave_sums4(v4, bz);
    const double s00 = 1.0 - bz[0], s01 = -bz[1], s10 = -bz[2], s11 = 1.0 - bz[3];
    const double g_e = a.gbar[2 * pt], g_y = a.gbar[2 * pt + 1];
    const double r0 = g_y, r1 = -g_e;  // dL/dYe, dL/de
    const double idet = 1.0 / (s00 * s11 - s01 * s10);
    const double l0 = (s11 * r0 - s01 * r1) * idet;
    const double l1 = (s00 * r1 - s10 * r0) * idet;
    double gq = 0.0, v2[4] = {0.0, 0.0, 0.0, 0.0};
    if (lane < 32) {
#pragma unroll
      for (int t = 0; t < NS; ++t) {
        const double lam = -(S.z0[t][q] * l0 + S.z1[t][q] * l1);
        gq -= lam * S.ds[t][q];
        v2[0] -= lam * S.da[t][q];
        v2[1] -= lam * S.dp[t][q];
      }
    }
    double gs[4];
    wave_sums4(v2, gs);
    const double nan = __builtin_nan("");
    g_s = ok ? gq : nan;
    g_nes = ok ? gs[0] : nan;
    g_pair = ok ? gs[1] : nan;
    __syncthreads();
  }
};

template <int NS>
struct AdjPairLds {
  ModelLds m;
  double row[5][NS][kLanes];  // dR_D / d(Ye, e, a_nes, a_pair, s_q) of the lane's rows
};

// most iterations before a point is left to the elimination, and the relative
// change of an entry at which it has settled (16 ulp; the next iteration
// would change it by a fraction of that)
constexpr int kAdjMaxIt = 24;
constexpr double kAdjSettled = 0x1p-48;
// bits that the largest change has to lose per iteration.  48 / kAdjMaxIt = 2
// would keep every point that can settle: 4-8% less for 65536 points of which a
// part settles slowly, but 8 points of the dense centre at 0.5 km then take 82 us
// instead of 54, a wavefront waiting for the slowest of them
constexpr int kAdjPace = 3;

// Two points per wavefront by iteration: lane 32 h + q holds node q of the
// point of half h, for every species.
//
// The contractions run on the symmetric core B2 = exp(-|e_q - e_p| / T) as in
// the forward kernel (columns broadcast by DPP, the other 16-lane row's share
// by one coefficient and one exchange, the factors g, 1 / g and h of the nodes
// on the vectors and the row sums).  Elimination alone is a chain of pivot
// broadcasts and reciprocals, 1488 us for 65536 points of the radial profile;
// with iterations over whole rows of 32 columns 324 us.  The narrower rows take
// forward solve and gradient together from 872 to 672 us.  The multiply-adds'
// issue at two waves per SIMD bounds it, a third of them the rates and their
// derivatives.
template <int NS>
struct PairAdjoint {
  // s[t] = sum_j B2(q, j) x_j[t] and d[t] = sum_j B2(q, j) f(q, j) x_j[t],
  // f(q, j) = fj(j) over this row's columns.  f is linear in e_q and e_j on
  // either side of the diagonal, so over the other row's columns it is
  // f(b, j) + f1 with b the node of that row next to this one
  // (Fmac4 takes four columns at a time).
  template <class F>
  __device__ __forceinline__ static void contract2(const double (&x)[NS], const double (&B)[16], double k, double f1,
                                                   double (&s)[NS], double (&d)[NS], F&& fj) {
#pragma unroll
    for (int t = 0; t < NS; ++t) s[t] = d[t] = 0.0;
    static_for<0, 4>([&](auto jj) __attribute__((always_inline)) {
      constexpr int j = 4 * decltype(jj)::value;
      Fmac4<NS>::template run<j>(s, d, x, B[j], B[j + 1], B[j + 2], B[j + 3], fj(j), fj(j + 1), fj(j + 2), fj(j + 3));
    });
    const bool upper = threadIdx.x & 16;
#pragma unroll
    for (int t = 0; t < NS; ++t) {
      const double ms = mirror32(s[t]), md = mirror32(d[t]);
      const double zs = upper ? row_bcast<0>(ms) : row_bcast<15>(ms), zd = upper ? row_bcast<0>(md) : row_bcast<15>(md);
      s[t] = __builtin_fma(k, zs, s[t]);
      d[t] = __builtin_fma(k, __builtin_fma(f1, zs, zd), d[t]);
    }
  }

  // live: the half's point has terms (solved forward, not skipped).  Returns
  // in every lane whether its half's point was solved here; g_s is the lane's
  // s_q term, g_nes and g_pair the point's.
  __device__ __forceinline__ static bool run(const AdjArgs& a, int64_t pt, bool live, AdjPairLds<NS>& S, double& g_s,
                                             double& g_nes, double& g_pair) {
    const_ptr<DevModel> md = scalar_ptr(a.mdl);
    const int lane = opaque((int)threadIdx.x);
    const int h = lane >> 5, q = lane & 31;
    const int64_t base = pt * (int64_t)(NS * NQ);
    double D[NS];
#pragma unroll
    for (int t = 0; t < NS; ++t) D[t] = a.D[base + md->ext[t] * NQ + q];
    const double rho = a.rho11[pt], ye = a.ye[pt], e = a.e[pt];
    const double chi0 = a.chi0 ? a.chi0[pt] : md->chi_ref * rho;
    const double dtau = a.dtau;
    // EOS and its derivatives
    const double r3 = cbrt(rho), cye = cbrt(ye);
    const double ia = rcp_nr(md->eos_a * (1.0 + ye));
    const double T = (e - md->eos_b * (ye * cye) * r3) * ia;
    const bool warm = live && T > 0.0 && isfinite(T);
    const double Tu = warm ? T : 1.0;
    const double mu = md->mu_a * (ye - md->mu_ye0) * r3 + md->mu_b * log_pos(Tu * md->inv_mu_t0);
    const double invT = rcp_nr(Tu);
    const double dT_de = ia;
    const double dT_dye = -(4.0 / 3.0) * md->eos_b * cye * r3 * ia - T * rcp_nr(1.0 + ye);
    const double dmu_dye = md->mu_a * r3 + md->mu_b * invT * dT_dye;
    const double dmu_de = md->mu_b * invT * dT_de;
    const double K = md->kcoup * rcp_nr(rho);
    const unsigned flags = md->flags;
    const double a_nes = (flags & NMC_NES) ? S.m.theta[NQ] : 0.0;
    const double a_pair = (flags & NMC_PAIR) ? S.m.theta[NQ + 1] : 0.0;

    // rows of the symmetric core and the nodes' factors (scaled by 2^+-c, c
    // the middle of the point's exponent range)
    const double eq = S.m.eps[q], w2q = S.m.w2[q], weq = w2q * eq;
    const ExpSplit xs = exp_split(eq, invT);
    const int lo0 = __builtin_amdgcn_readlane(xs.n, 0), hi0 = __builtin_amdgcn_readlane(xs.n, 31);
    const int lo1 = __builtin_amdgcn_readlane(xs.n, 32), hi1 = __builtin_amdgcn_readlane(xs.n, 63);
    const int nlo = h ? lo1 : lo0, nhi = h ? hi1 : hi0;
    const int c = (nlo + nhi) >> 1;
    bool act = warm && nhi - nlo <= pairk::kDirectBits;
    if (__builtin_amdgcn_ballot_w64(act) == 0) return false;
    const double gq = ldexp(xs.R, c - xs.n), rgq = ldexp(xs.P, xs.n - c);
    const double hq = ldexp(xs.R * xs.R, -2 * xs.n);  // exp(-e / T)
    double B[16], kx;
    pairk::direct_row_regs(gq * gq, rgq * rgq, B, kx);

    // ---- rates with unit-amplitude kernels, their temperature derivatives
    // (times T^2) and the rows of dR_D / d(Ye, e, a_nes, a_pair, s_q) -------
    double dg[NS], c0[NS], c1[NS];  // diagonal of A^T, right-hand sides over it
    {
      double x[NS], en[NS], dn[NS], on[NS], dout[NS], an[NS], dan[NS], ep[NS], dpr[NS];
      // d = e_q - e_j over this row and its magnitude; e_q is laundered
      // between the passes, so that they are formed again instead of held
      const int r16 = q & 16;
      double ev = eq;
      auto dl = [&](int j) { return ev - S.m.eps[r16 + j]; };
      auto ad = [&](int j) { return fabs(dl(j)); };
      const double eb = eq - S.m.eps[r16 ? 15 : 16];  // from the other row's node next to this row
#pragma unroll
      for (int t = 0; t < NS; ++t) x[t] = weq * D[t] * rgq;
      contract2(x, B, kx, __builtin_fma(0.5, eb, fabs(eb)), en, dn,
                [&](int j) { return B[j] * __builtin_fma(0.5, dl(j), ad(j)); });
      asm volatile("" : "+v"(ev));
#pragma unroll
      for (int t = 0; t < NS; ++t) x[t] = weq * (1.0 - D[t]) * gq;
      contract2(x, B, kx, __builtin_fma(-0.5, eb, fabs(eb)), on, dout,
                [&](int j) { return B[j] * __builtin_fma(-0.5, dl(j), ad(j)); });
      asm volatile("" : "+v"(ev));
#pragma unroll
      for (int t = 0; t < NS; ++t) x[t] = weq * D[pair_partner<NS>(t)];
      contract2(x, B, kx, fabs(eb), an, dan, [&](int j) { return B[j] * ad(j); });
      asm volatile("" : "+v"(ev));
#pragma unroll
      for (int t = 0; t < NS; ++t) x[t] = weq * (1.0 - D[pair_partner<NS>(t)]) * hq;
      contract2(x, B, kx, fabs(eb) + eb, ep, dpr, [&](int j) { return B[j] * (ad(j) + (ev + S.m.eps[r16 + j])); });
      const double sc = rho * eq, scg = sc * gq, scr = sc * rgq, sch = sc * hq;
      const double shape = chi0 * S.m.shape[q], iT2 = invT * invT;
      const double wen = dtau * a_nes * sc * weq, wep = dtau * a_pair * sc * weq;
#pragma unroll
      for (int t = 0; t < NS; ++t) {
        en[t] *= scg;
        dn[t] *= scg;
        on[t] *= scr;
        dout[t] *= scr;
        an[t] *= sc;
        dan[t] *= sc;
        ep[t] *= sch;
        dpr[t] *= sch;
        const double chia = (flags & NMC_EMAB) ? md->iemab[t] * S.m.theta[q] * shape : 0.0;
        const double xf = (eq - md->imusign[t] * mu) * invT;
        const double ex = exp(-fabs(xf));
        const double r = rcp_nr(1.0 + ex);
        const double f = xf > 0.0 ? ex * r : r;   // Fermi-Dirac D_eq
        const double fc = xf > 0.0 ? r : ex * r;  // 1 - D_eq
        const double ddeq_dT = f * fc * xf * invT;
        const double ddeq_dmu = f * fc * md->imusign[t] * invT;
        const double chi = chia + a_nes * (en[t] + on[t]) + a_pair * (ep[t] + an[t]);
        const double deta_dT = chia * ddeq_dT + (a_nes * dn[t] + a_pair * dpr[t]) * iT2;
        const double dchi_dT = (a_nes * (dn[t] + dout[t]) + a_pair * (dpr[t] + dan[t])) * iT2;
        const double dR_dT = dtau * (D[t] * dchi_dT - deta_dT);
        const double dR_dmu = -dtau * chia * ddeq_dmu;
        S.row[0][t][lane] = dR_dT * dT_dye + dR_dmu * dmu_dye;
        S.row[1][t][lane] = dR_dT * dT_de + dR_dmu * dmu_de;
        S.row[2][t][lane] = (flags & NMC_NES) ? dtau * (D[t] * (en[t] + on[t]) - en[t]) : 0.0;
        S.row[3][t][lane] = (flags & NMC_PAIR) ? dtau * (D[t] * (ep[t] + an[t]) - ep[t]) : 0.0;
        S.row[4][t][lane] = (flags & NMC_EMAB) ? dtau * shape * md->iemab[t] * (D[t] - f) : 0.0;
        // the diagonal entry: NES self term Phi_in[q][q] = Phi_out[q][q] = A e^2, and for a species that is its own
        // pair partner the pair term of Phi_ann[q][q] = A' e^2, Phi_pro[q][q] = A' e^2 h^2
        double diag = 1.0 + dtau * chi - wen;
        if (pair_partner<NS>(t) == t) diag += wep * (D[t] + (1.0 - D[t]) * (hq * hq));
        dg[t] = diag;
        const double rd = rcp_nr(diag);
        c0[t] = K * md->ig[t] * w2q * rd;
        c1[t] = K * md->imult[t] * S.m.w3[q] * rd;
      }
    }

    // ---- z <- (c + (G - A^T) z) / G for both right-hand sides --------------
    // (A^T z)_q = G z + the NES sum over the own species and the pair sum over
    // the partner, with the diagonal terms taken out again
    double z[2][NS];
#pragma unroll
    for (int t = 0; t < NS; ++t) {
      z[0][t] = c0[t];
      z[1][t] = c1[t];
    }
    bool solved = false;
    const double wn = dtau * a_nes * rho * weq, wp = dtau * a_pair * rho * weq;
    for (int it = 0; it < kAdjMaxIt && __builtin_amdgcn_ballot_w64(act) != 0; ++it) {
#pragma unroll
      for (int j = 0; j < 16; ++j) asm volatile("" : "+v"(B[j]));
      // after 2, 6 and 12 iterations the changes have to be down to pace
      const int done = it + 1;
      const bool look = done == 2 || done == 6 || done == 12;
      const double pace = ldexp(1.0, 1 - kAdjPace * done);
      bool moved = false, behind = false;
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        double xg[NS], yg[NS], xd[NS], hy[NS];
#pragma unroll
        for (int t = 0; t < NS; ++t) {
          const double ez = eq * z[k][t];
          xd[t] = ez * D[t];
          const double yd = ez - xd[t];
          xg[t] = xd[t] * rgq;
          yg[t] = yd * gq;
          hy[t] = yd * hq;
        }
        double eN[NS], oN[NS], aP[NS], eP[NS];
        pairk::core_contract<NS>(B, kx, xg, yg, xd, hy, eN, oN, aP, eP);
#pragma unroll
        for (int t = 0; t < NS; ++t) {
          const double ez = eq * z[k][t];
          // the sums without their q-th terms, B2(q, q) = 1
          double nes = __builtin_fma(gq, eN[t], rgq * oN[t]) - ez;
          double pr = __builtin_fma(hq, eP[t], aP[t]);
          if (pair_partner<NS>(t) == t) pr -= ez * __builtin_fma(1.0 - D[t], hq * hq, D[t]);
          const double off = __builtin_fma(wn, nes, -wp * pr);
          const double cc = k ? c1[t] : c0[t];
          const double zn = __builtin_fma(off, rcp_nr(dg[t]), cc);
          const double change = fabs(zn - z[k][t]), size = fabs(zn) + fabs(cc);
          moved = moved || !(change <= kAdjSettled * size);
          if (look) behind = behind || !(change <= pace * size);
          z[k][t] = act ? zn : z[k][t];
        }
      }
      const bool on = pairk::half_any(moved);
      solved = solved || (act && !on);
      act = act && on && !pairk::half_any(behind);
    }

    // ---- Schur complement on (Ye, e), multipliers and gradient ------------
    double v4[4] = {0.0, 0.0, 0.0, 0.0}, bz[4];
#pragma unroll
    for (int t = 0; t < NS; ++t) {
      const double b0 = S.row[0][t][lane], b1 = S.row[1][t][lane];
      v4[0] += b0 * z[0][t];
      v4[1] += b0 * z[1][t];
      v4[2] += b1 * z[0][t];
      v4[3] += b1 * z[1][t];
    }
    pairk::half_sums4(v4, bz);
    const double s00 = 1.0 - bz[0], s01 = -bz[1], s10 = -bz[2], s11 = 1.0 - bz[3];
    const double g_e = a.gbar[2 * pt], g_y = a.gbar[2 * pt + 1];
    const double r0 = g_y, r1 = -g_e;  // dL/dYe, dL/de
    const double idet = 1.0 / (s00 * s11 - s01 * s10);
    const double l0 = (s11 * r0 - s01 * r1) * idet;
    const double l1 = (s00 * r1 - s10 * r0) * idet;
    double v2[2] = {0.0, 0.0}, gs[2];
    g_s = 0.0;
#pragma unroll
    for (int t = 0; t < NS; ++t) {
      const double lam = z[0][t] * l0 + z[1][t] * l1;  // -lambda
      g_s += lam * S.row[4][t][lane];
      v2[0] += lam * S.row[2][t][lane];
      v2[1] += lam * S.row[3][t][lane];
    }
    pairk::half_own_sums<1>(v2, gs);
    g_nes = gs[0];
    g_pair = gs[1];
    return solved;
  }
};

// What a work-group adds up: the terms of the points of each half, the lane's
// node and the two amplitudes
struct AdjSums {
  double s = 0.0, nes = 0.0, pair = 0.0;
  // the work-group's row of partial sums
  __device__ __forceinline__ void store(double* __restrict__ row) const {
    const int lane = threadIdx.x;
    const double a = sum_halves(s), b = sum_halves(nes), c = sum_halves(pair);
    const double v = lane < NQ ? a : (lane == NQ ? b : c);
    if (lane < NQ + 2) row[lane] = v;
  }
};

// the terms of point pt, one lane half's worth, to the caller's array
__device__ __forceinline__ void store_terms(double* grad_pp, int64_t pt, double s, double nes, double pair) {
  const int q = threadIdx.x & 31;
  double* gout = grad_pp + pt * (NQ + 2);
  gout[q] = s;
  if (q < 2) gout[NQ + q] = q ? pair : nes;
}

template <int NS>
__global__ __launch_bounds__(kLanes, 2) void adj_kernel(AdjArgs a) {
  __shared__ AdjPairLds<NS> S;
  load_model(a.mdl, a.theta, S.m);
  const int lane = threadIdx.x, h = lane >> 5;
  AdjSums sum;
  const int64_t pairs = (a.P + 1) / 2;
  for (int64_t u = blockIdx.x; u < pairs; u += gridDim.x) {
    // past the end of an odd batch the half mirrors its neighbour and counts for nothing
    const int64_t raw = 2 * u + h;
    const bool has_point = raw < a.P;
    const int64_t pt = has_point ? raw : raw - 1;
    // skipped or failed points contribute nothing
    const bool live = has_point && a.status[pt] == NMC_STATUS_OK && a.n_outer[pt] != 0;
    double g_s = 0.0, g_nes = 0.0, g_pair = 0.0;
    uint64_t left = 0;
    if (__builtin_amdgcn_ballot_w64(live) != 0) {
      const bool solved = PairAdjoint<NS>::run(a, pt, live, S, g_s, g_nes, g_pair);
      if (!solved) g_s = g_nes = g_pair = 0.0;
      left = __builtin_amdgcn_ballot_w64(live && !solved);
    }
    sum.s += g_s;
    sum.nes += g_nes;
    sum.pair += g_pair;
    if (a.grad_pp && has_point) store_terms(a.grad_pp, pt, g_s, g_nes, g_pair);
    if (lane == 0) a.left[u] = (uint8_t)((left & 1) | ((left >> 32) & 1) << 1);
    __syncthreads();
  }
  sum.store(a.partial + (int64_t)blockIdx.x * (NQ + 2));
}

// The points that the iteration left over, by elimination: every work-group
// looks through the flags of its own points, 64 at a time, and writes a row of
// partial sums if it had any, so the order of the sums is fixed.
template <int NS>
__global__ __launch_bounds__(kLanes) void adj_left_kernel(AdjArgs a) {
  __shared__ AdjLds<NS> S;
  const int lane = threadIdx.x, h = lane >> 5;
  AdjSums sum;
  bool any = false;
  for (int64_t p0 = blockIdx.x; p0 < a.P; p0 += (int64_t)kLanes * gridDim.x) {
    const int64_t p = p0 + (int64_t)lane * gridDim.x;
    const bool mine = p < a.P && ((a.left[p >> 1] >> (p & 1)) & 1) != 0;
    for (uint64_t todo = __builtin_amdgcn_ballot_w64(mine); todo != 0; todo &= todo - 1) {
      if (!any) load_model(a.mdl, a.theta, S.m);
      any = true;
      const int64_t pt = uniform64(p0 + (int64_t)__builtin_ctzll(todo) * gridDim.x);
      double g_s, g_nes, g_pair, own, other;
      PointAdjoint<NS>::run(a, pt, S, g_s, g_nes, g_pair);
      swap32(g_s, own, other);  // the s_q terms of lanes 0..31 in both halves
      sum.s += h == 0 ? own : 0.0;
      sum.nes += h == 0 ? g_nes : 0.0;
      sum.pair += h == 0 ? g_pair : 0.0;
      if (a.grad_pp && h == 0) store_terms(a.grad_pp, pt, own, g_nes, g_pair);
    }
  }
  if (any) sum.store(a.partial_left + (int64_t)blockIdx.x * (NQ + 2));
  if (lane == 0) a.had[blockIdx.x] = any ? 1 : 0;
}

template <int NS>
void launch_adjoint_t(const AdjArgs& a, unsigned grid, unsigned grid_left, hipStream_t s) {
  hipLaunchKernelGGL(adj_kernel<NS>, dim3(grid), dim3(kLanes), 0, s, a);
  hipLaunchKernelGGL(adj_left_kernel<NS>, dim3(grid_left), dim3(kLanes), 0, s, a);
}

// Adds the work-groups' rows of partial sums to out, one work-group per
// column: thread t adds rows t, t + 256, ... of the iteration in order, then
// rows 16 t .. 16 t + 15 of the elimination where they are marked, then a
// fixed-shape tree over the 256 threads.  (One work-group for all 34 columns
// took 55 us.)
__global__ __launch_bounds__(256) void reduce_partials(AdjArgs a, int rows, int rows_left, int ncol,
                                                       double* __restrict__ out) {
  __shared__ double red[256];
  const int t = threadIdx.x, c = blockIdx.x;
  double s = 0.0;
  for (int b = t; b < rows; b += 256) s += a.partial[(int64_t)b * ncol + c];
  static_assert(kAdjPartials == 256 * 16, "16 marks per thread");
  const uint4 had = ((const uint4*)a.had)[t];
  if ((had.x | had.y | had.z | had.w) != 0) {
    const uint32_t word[4] = {had.x, had.y, had.z, had.w};
    for (int i = 0; i < 16; ++i) {
      const int b = 16 * t + i;
      if (b < rows_left && (word[i >> 2] >> (8 * (i & 3)) & 0xff) != 0) s += a.partial_left[(int64_t)b * ncol + c];
    }
  }
  red[t] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (t < w) red[t] += red[t + w];
    __syncthreads();
  }
  if (t == 0) out[c] += red[0];
}

}  // namespace

hipError_t launch_adjoint(const AdjArgs& a, int nq, int ns, int num_cu, double* grad_theta, hipStream_t s) {
  if (nq != NQ || ns < 1 || ns > 3) return hipErrorInvalidValue;
  if (a.P == 0) return hipSuccess;
  const AdjGrid g = adj_grid(a.P, num_cu);
  const unsigned grid = (unsigned)g.iterate, left = (unsigned)g.eliminate;
  switch (ns) {
    case 1: launch_adjoint_t<1>(a, grid, left, s); break;
    case 2: launch_adjoint_t<2>(a, grid, left, s); break;
    default: launch_adjoint_t<3>(a, grid, left, s); break;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(reduce_partials, dim3(NQ + 2), dim3(256), 0, s, a, (int)grid, (int)left, NQ + 2, grad_theta);
  return hipGetLastError();
}

}  // namespace nmc
