// Forward kernel of the O(v) coupling solve for 32 energy nodes and small
// batches: one work-group per pair of points, one wavefront per species
// (CDNA4).
//
// The decomposition of the static small-batch kernel (nmc_forward_split.hip)
// with the equations of the two-point O(v) kernel: wave t holds the four
// moments (D, I_1, I_2, I_3) of species t of both points, lane 32 h + q node q
// of the point of half h.  A wave of the two-point kernel needs more than 256
// registers for three species (one wave per SIMD, its dependent chains
// exposed) and ~1120 instructions per inner iteration; a species' share fits
// two waves per SIMD with its Anderson history in registers and takes ~430.
// Through LDS go the lane's terms of the Gram sums of the Anderson step, the
// moments of the pair partner and the convergence flags (two barriers per inner
// iteration) and the lane's terms of the Eulerian integrals of the matter
// update.  What follows from them is computed by every wave from the same
// values, so the waves take every branch together.  Sums over species add the lane's terms in
// the two-point kernel's order and the sums of one species take its reduction
// tree, so the two kernels give the same bits.
#include "nmc_closure.h"
#include "nmc_split.h"

namespace nmc {
namespace {

using namespace pairk;
using namespace splitk;

constexpr double kMuC2s = 931.49410242;  // atomic mass unit rest energy [MeV]

template <int NS, bool PHI1>
struct VSplitLds {
  ModelLds m;
  SplitExp E[2];                       // per point: exponent splits (points too cold for scaled factors)
  double M[NS][PHI1 ? 4 : 1][kLanes];  // next moments of every species (the flux for the linear-order terms)
  alignas(16) double gram[NS][kLanes][4];   // the lane's terms of the Gram sums of the Anderson step
  double X[NS][5][kLanes];                  // the lane's terms of the Eulerian integrals (N, E, F_1, F_2, F_3)
  int flag[NS][2];           // 1: converged, 2: a non-finite iterate
  struct Pt {                // state of the outer (matter) loop: every wave keeps its own copy
    double y[5], yst[5], yused[5], X0[5];
    double oq[5], of[5], odq[5], odf[5];
  } pt[NS][2];
};

template <int NS, bool PHI1>
struct VSplitSolver {
  static constexpr int NQ = NQP;
  using Lds = VSplitLds<NS, PHI1>;
  using Pt = typename Lds::Pt;

  __device__ __forceinline__ static double temperature(const_ptr<DevModel> md, const double* y, double r3) {
    const double v2 = y[2] * y[2] + y[3] * y[3] + y[4] * y[4];
    const double e = y[1] - 0.5 * kMuC2s * v2;
    return (e - md->eos_b * ye43(y[0]) * r3) * rcp_nr(md->eos_a * (1.0 + y[0]));
  }

  // Eulerian integrals (N, E, F_1, F_2, F_3) of the half's point at velocity
  // v, in every lane; one form for every caller, so that equal moments give
  // bitwise equal integrals
  __device__ __forceinline__ static void eulerian(Lds& S, const_ptr<DevModel> md, int sp, int lane, int q, double D,
                                                  const double (&I)[3], const double (&v)[3], double (&X)[5]) {
    const double w2 = S.m.w2[q], w3 = S.m.w3[q];
    double vI, vK[3];
    closure_terms_flat(D, I, v, vI, vK);
    __syncthreads();  // the last terms have been read
    S.X[sp][0][lane] = D + vI;
    S.X[sp][1][lane] = D + 2.0 * vI;
#pragma unroll
    for (int j = 0; j < 3; ++j) S.X[sp][2 + j][lane] = I[j] + v[j] * D + vK[j];
    __syncthreads();
    double acc[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0}, s[6];
#pragma unroll
    for (int t = 0; t < NS; ++t) {
      acc[0] += md->ig[t] * w2 * S.X[t][0][lane];
#pragma unroll
      for (int i = 1; i < 5; ++i) acc[i] += md->imult[t] * w3 * S.X[t][i][lane];
    }
    half_own_sums<3>(acc, s);
#pragma unroll
    for (int i = 0; i < 5; ++i) X[i] = s[i];
  }

  // matter right-hand side q(M, y) of Eq. implicitFluidNodal from the
  // integrals X of the current moments
  __device__ __forceinline__ static void matter_rhs(const Pt& pt, double K, const double (&X)[5], double (&yq)[5]) {
    yq[0] = pt.yst[0] - K * (X[0] - pt.X0[0]);
    yq[1] = pt.yst[1] - K * (X[1] - pt.X0[1]);
    const double Kv = K * (1.0 / kMuC2s);
#pragma unroll
    for (int j = 0; j < 3; ++j) yq[2 + j] = pt.yst[2 + j] - Kv * (X[2 + j] - pt.X0[2 + j]);
  }

  __device__ __forceinline__ static void solve(int64_t u, Lds& S) {
    const_ptr<FwdVArgs> a = kernel_args<FwdVArgs>();
    const DevModel* mdl = a->mdl;
    const_ptr<DevModel> md = scalar_ptr(mdl);
    const ModelLds& mt = S.m;
    const int sp = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // this wave's species (internal order)
    const int pa = NS == 3 ? (sp < 2 ? 1 - sp : 2) : 1 - sp;          // its pair partner
    const int lane = threadIdx.x & 63;
    const int h = lane >> 5, q0 = lane & 31;
    const double dtau = a->dtau;
    // point of this half; past the end of an odd batch the half mirrors its
    // neighbour and stores nothing
    const int64_t p_raw = 2 * u + h;
    const bool has_point = p_raw < a->P;
    const int64_t p = has_point ? p_raw : p_raw - 1;
    const int ex = md->ext[sp];
    const int64_t oD = (p * NS + ex) * (int64_t)NQ + q0, oI = (p * NS + ex) * (int64_t)(3 * NQ) + q0;
    const double rho = in_global(a->rho11)[p];
    Pt& pt = S.pt[sp][h];

    double D = in_global(a->D0)[oD], I[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) I[j] = in_global(a->I0)[oI + j * NQ];
    double yst[5];
    yst[0] = in_global(a->ye0)[p];
    yst[1] = in_global(a->ef0)[p];
#pragma unroll
    for (int j = 0; j < 3; ++j) yst[2 + j] = in_global(a->v0)[3 * p + j];
    S.M[sp][0][lane] = D;
    if constexpr (PHI1) {
#pragma unroll
      for (int j = 0; j < 3; ++j) S.M[sp][1 + j][lane] = I[j];
    }

    // coupling disabled at low density (Sec. 7.2): the state passes through
    const bool skip = rho < md->rho11_min;
    const double r3 = cbrt(rho), K = md->kcoup / rho;
    const double An = (md->flags & NMC_NES) ? mt.theta[NQ] * rho : 0.0;
    const double Ap = (md->flags & NMC_PAIR) ? mt.theta[NQ + 1] * rho : 0.0;
    const double chi0 = a->chi0 ? in_global(a->chi0)[p] : md->chi_ref * rho;
#pragma unroll
    for (int i = 0; i < 5; ++i) {
      pt.yst[i] = pt.y[i] = pt.yused[i] = yst[i];
      pt.oq[i] = pt.of[i] = pt.odq[i] = pt.odf[i] = 0.0;
    }
    double T_last = temperature(md, yst, r3);

    // old conserved moments N* = D* + v*.I*, G*_j = I*_j + v*^i K*_ij, the old
    // Eulerian integrals and ||D*||_W^2
    double Nst, Gst[3];
    auto norm = [&](double w2) {
      const double v[2] = {w2 * D * D, 0.0};
      double s[2];
      half_own_sums<1>(v, s);
      return s[0];
    };
    double dref = norm(mt.w2[q0]);
    {
      const double vs[3] = {yst[2], yst[3], yst[4]};
      double vI, vK[3], X0[5];
      closure_terms(D, I, vs, vI, vK);
      Nst = D + vI;
#pragma unroll
      for (int j = 0; j < 3; ++j) Gst[j] = I[j] + vK[j];
      eulerian(S, md, sp, lane, q0, D, I, vs, X0);
#pragma unroll
      for (int i = 0; i < 5; ++i) pt.X0[i] = X0[i];
    }
    // moments of the partner (the barriers above have passed)
    double Dp = S.M[pa][0][lane], Ip[PHI1 ? 3 : 1];
    if constexpr (PHI1) {
#pragma unroll
      for (int j = 0; j < 3; ++j) Ip[j] = S.M[pa][1 + j][lane];
    }
    __syncthreads();

    int status = NMC_STATUS_OK;
    bool fatal = false, inner_failed = false, outer_conv = false;
    bool run = !skip;  // this half's point is still iterating the outer loop
    int k_done = 0, total_inner = 0;

    for (int k = 1; k <= a->prm.max_outer && __builtin_amdgcn_ballot_w64(run) != 0; ++k) {
      const_ptr<FwdVArgs> a = kernel_args<FwdVArgs>();
      const_ptr<DevModel> md = scalar_ptr(mdl);
      const int q = opaque(q0);
      if (run) k_done = k;
      // ---- ComputeOpacities(y^[k]) --------------------------------------
      const double v[3] = {pt.y[2], pt.y[3], pt.y[4]};
      const double lam = rcp_nr(1.0 + sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]));
      const double T = temperature(md, a->prm.fixed_matter ? pt.yst : pt.y, r3);
      const double y0 = pt.y[0];
      const double mu = md->mu_a * (y0 - md->mu_ye0) * r3 + md->mu_b * log_pos(T * md->inv_mu_t0);
      if (run && (!(T > 0.0) || !(y0 >= 0.0) || !isfinite(T) || !isfinite(mu))) {
        status = NMC_STATUS_EOS_DOMAIN;
        fatal = true;
        run = false;
      }
      if (run) {
        T_last = T;
#pragma unroll
        for (int i = 0; i < 5; ++i) pt.yused[i] = pt.y[i];
      }
      // a finished half keeps a harmless temperature
      const double Tu = run ? T : 1.0, muu = run ? mu : 0.0;
      const double invT = rcp_nr(Tu);
      const double ldt = lam * dtau, oml = 1.0 - lam;
      const double epsq = mt.eps[q];
      const ExpSplit xs = exp_split(epsq, invT);
      // lam (N* + dtau chi^EmAb D_eq), 1 + lam dtau chi^EmAb and 1 + lam dtau (chi^EmAb + sigma)
      const double shape = chi0 * mt.shape[q];
      const double sig = (md->flags & NMC_ISO) ? md->sigma_ratio * shape : 0.0;
      const double chia = md->iemab[sp] * ((md->flags & NMC_EMAB) ? mt.theta[q] * shape : 0.0);
      const double xf = (epsq - md->imusign[sp] * muu) * invT;
      const double exf = exp(-fabs(xf));
      const double rf = rcp_nr(1.0 + exf);
      const double deq = xf > 0.0 ? exf * rf : rf;
      const double baseD = lam * (Nst + dtau * (chia * deq));
      const double denD = 1.0 + ldt * chia, denI = 1.0 + ldt * (chia + sig);

      // row of the symmetric core with the nodes' factors g and 1 / g scaled
      // by 2^+-c (every wave of the work-group forms the same row), where the
      // grid spans at most kDirectBits powers of two; else from the exponent
      // splits in LDS (cold_rows), signed beyond kSymBits
      double B[16], kx, gq = 1.0, rgq = 1.0;
      const double hq = ldexp(xs.R * xs.R, -2 * xs.n);  // exp(-e / T)
      const int lo0 = __builtin_amdgcn_readlane(xs.n, 0), hi0 = __builtin_amdgcn_readlane(xs.n, 31);
      const int lo1 = __builtin_amdgcn_readlane(xs.n, 32), hi1 = __builtin_amdgcn_readlane(xs.n, 63);
      const int nlo = h ? lo1 : lo0, nhi = h ? hi1 : hi0;
      const int c = (nlo + nhi) >> 1;
      const bool direct = __builtin_amdgcn_ballot_w64(run && nhi - nlo > kDirectBits) == 0;
      const bool sym = __builtin_amdgcn_ballot_w64(run && nhi - nlo > kSymBits) == 0;
      if (sym) {
        gq = ldexp(xs.R, c - xs.n);
        rgq = ldexp(xs.P, xs.n - c);
      }
      if (direct) {
        direct_row_regs(gq * gq, rgq * rgq, B, kx);
      } else if (sym) {
        cold_rows<true>(S.E[h], q, xs, B, kx);
      } else {
        cold_rows<false>(S.E[h], q, xs, B, kx);
      }

      // ---- inner loop over moments at fixed matter (M^[k,1] = M^[k-1,*]) --
      const double w2q = mt.w2[q], w2eq = w2q * epsq;
      const double Aeq = An * epsq, Apq = Ap * epsq, Apqh = Apq * hq;
      const double ag = Aeq * gq, arg = Aeq * rgq;
      double G11 = 0.0;
      double Qp[4], Fp[4], dQo[4], dFo[4];  // Anderson history
#pragma unroll
      for (int x = 0; x < 4; ++x) Qp[x] = Fp[x] = dQo[x] = dFo[x] = 0.0;
      const double dref0 = dref;
      const bool ran = run;
      bool act = run;
      bool cvd = false;
      int l_done = 0;
      const int m_inner = held(a->prm.m_inner), max_inner = held(a->prm.max_inner);
      const double tol2 = held(a->tol_inner2);
      for (int l = 1; l <= max_inner && __builtin_amdgcn_ballot_w64(act) != 0; ++l) {
        if (act) l_done = l;
#pragma unroll
        for (int j = 0; j < 16; ++j) asm volatile("" : "+v"(B[j]));
        double etaN[1], outN[1], annP[1], etaP[1];
        {
          const double xv = w2eq * D, yv = w2eq - xv;
          const double xp[1] = {w2eq * Dp}, hyp[1] = {hq * (w2eq - xp[0])};
          if (sym) {
            const double xg[1] = {xv * rgq}, yg[1] = {yv * gq};
            core_contract<1>(B, kx, xg, yg, xp, hyp, etaN, outN, annP, etaP);
          } else {
            signed_split(B, kx, xv, yv, xp[0], hyp[0], etaN[0], outN[0], annP[0], etaP[0]);
          }
        }
        // linear-order corrections at the current iterate (see the two-point kernel)
        double cN = 0.0, cI[3] = {0.0, 0.0, 0.0};
        if constexpr (PHI1) {
          const double rN = md->phi1_nes * Aeq, rP = md->phi1_pair * Apq;
          double Pc[3], Rc[3];
#pragma unroll
          for (int i = 0; i < 3; ++i) {
            const double x = w2eq * I[i];
            double eN[1], oN[1], aP[1], eP[1];
            const double xp[1] = {w2eq * Ip[i]}, hxp[1] = {hq * xp[0]};
            if (sym) {
              const double xg[1] = {x * rgq}, yg[1] = {x * gq};
              core_contract<1>(B, kx, xg, yg, xp, hxp, eN, oN, aP, eP);
            } else {
              signed_split(B, kx, x, x, xp[0], hxp[0], eN[0], oN[0], aP[0], eP[0]);
            }
            Pc[i] = __builtin_fma(rN, gq * eN[0], -rP * (hq * eP[0]));
            Rc[i] = __builtin_fma(rN, rgq * oN[0], -rP * aP[0]);
          }
          phi1_collision_flat(D, I, Pc, Rc, cN, cI);
        }
        // Q and residual of the owned moments (Eq. implicitMomentsNodal); one
        // reciprocal of the product of the two denominators serves both
        double Q[4], F[4], Xn[4];
        {
          const double eta = __builtin_fma(ag, etaN[0], Apqh * etaP[0]);
          const double chi = __builtin_fma(arg, outN[0], __builtin_fma(Apq, annP[0], eta));
          double vI, vK[3];
          closure_terms_flat(D, I, v, vI, vK);
          const double dD = __builtin_fma(ldt, chi, denD), dI = __builtin_fma(ldt, chi, denI);
          const double r = rcp_nr(dD * dI);
          double nD = __builtin_fma(oml, D, baseD) - lam * vI + ldt * eta;
          if constexpr (PHI1) nD = __builtin_fma(ldt, cN, nD);
          Q[0] = nD * (r * dI);
#pragma unroll
          for (int j = 0; j < 3; ++j) {
            double nI = __builtin_fma(oml, I[j], lam * Gst[j]) - lam * vK[j];
            if constexpr (PHI1) nI = __builtin_fma(ldt, cI[j], nI);
            Q[1 + j] = nI * (r * dD);
          }
#pragma unroll
          for (int x = 0; x < 4; ++x) {
#pragma clang fp contract(off)
            F[x] = Q[x] - (x ? I[x ? x - 1 : 0] : D);  // from the rounded Q, not fused with its last product
          }
        }
        // Anderson step over min(l, M_inner) residuals (difference form)
        const int mem = l < m_inner ? l : m_inner;
        if (mem == 1) {
#pragma unroll
          for (int x = 0; x < 4; ++x) {
            Xn[x] = Q[x];
            dQo[x] = dFo[x] = 0.0;
          }
          __syncthreads();  // the flags and moments of the last iterate have been read
        } else {
          double p4[4], v4[4], gs[4];
#pragma unroll
          for (int x = 0; x < 4; ++x) {
            const double dF2 = F[x] - Fp[x];
            gram_terms(x, dFo[x], dF2, F[x], p4);
            dFo[x] = dF2;
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) S.gram[sp][lane][i] = p4[i];
          __syncthreads();
#pragma unroll
          for (int i = 0; i < 4; ++i) v4[i] = S.gram[0][lane][i];
#pragma unroll
          for (int t = 1; t < NS; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) v4[i] += S.gram[t][lane][i];
          half_sums4(v4, gs);
          double g1, g2;
          anderson2(mem == 3, G11, gs[0], gs[1], gs[2], gs[3], g1, g2);
#pragma unroll
          for (int x = 0; x < 4; ++x) {
#pragma clang fp contract(off)
            const double dQ2 = Q[x] - Qp[x];
            Xn[x] = __builtin_fma(-g1, dQo[x], __builtin_fma(-g2, dQ2, Q[x]));
            dQo[x] = dQ2;
          }
          G11 = gs[1];
        }
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          Qp[x] = Q[x];
          Fp[x] = F[x];
        }
        // Algorithm innerConverged over the four moments of this species
        // (compared squared), and whether an iterate is non-finite
        bool odd = false;
#pragma unroll
        for (int x = 0; x < 4; ++x) odd = odd || !isfinite(Xn[x]);
        const bool bad = half_any(odd, h);
        double vm[4], dm2, dn2;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const double d = Xn[x] - (x ? I[x ? x - 1 : 0] : D);
          vm[x] = w2q * d * d;
        }
        conv_sums(vm, w2q * Xn[0] * Xn[0], dm2, dn2);
        const bool conv1 = !half_any(!(dm2 <= tol2 * (dref0 > dn2 ? dref0 : dn2)), h);
        if (q0 == 0) S.flag[sp][h] = (conv1 ? 1 : 0) | (bad ? 2 : 0);
#pragma unroll
        for (int x = 0; x < (PHI1 ? 4 : 1); ++x) S.M[sp][x][lane] = Xn[x];
        __syncthreads();
        int all = 1, any = 0;
#pragma unroll
        for (int t = 0; t < NS; ++t) {
          all &= S.flag[t][h];
          any |= S.flag[t][h];
        }
        const double Dpn = S.M[pa][0][lane];
        double Ipn[PHI1 ? 3 : 1];
        if constexpr (PHI1) {
#pragma unroll
          for (int j = 0; j < 3; ++j) Ipn[j] = S.M[pa][1 + j][lane];
        }
        if ((any & 2) && act) {
          status = NMC_STATUS_NONFINITE;
          fatal = true;
          act = run = false;
        }
        if (act) {
          D = Xn[0];
#pragma unroll
          for (int j = 0; j < 3; ++j) I[j] = Xn[1 + j];
          Dp = Dpn;
          if constexpr (PHI1) {
#pragma unroll
            for (int j = 0; j < 3; ++j) Ip[j] = Ipn[j];
          }
          if (all & 1) {
            // ||D^[k,*]|| is the reference of the next inner loop
            dref = dn2;
            cvd = true;
            act = false;
          }
        }
      }
      if (ran) total_inner += l_done;
      if (run && !cvd) inner_failed = true;
      // the Eulerian integrals of the current moments at the matter iterate,
      // and after a failed loop the norm of the current moments
      if (__builtin_amdgcn_ballot_w64(run && !cvd) != 0) {
        const double n = norm(w2q);
        dref = (run && !cvd) ? n : dref;
      }
      double X[5];
      eulerian(S, md, sp, lane, q, D, I, v, X);
      if (a->prm.fixed_matter) {
        if (run) outer_conv = true;
        run = false;
      }
      if (run) {
        // ---- matter right-hand side, residual, outer Anderson step on y ----
        double yq[5], f[5], yn[5];
        matter_rhs(pt, K, X, yq);
#pragma unroll
        for (int i = 0; i < 5; ++i) f[i] = yq[i] - pt.y[i];
        const int omem = k < a->prm.m_outer ? k : a->prm.m_outer;
        if (omem == 1) {
#pragma unroll
          for (int i = 0; i < 5; ++i) yn[i] = yq[i];
        } else {
          double dq2[5], df2[5];
          double G22 = 0.0, b2 = 0.0, G11o = 0.0, G12 = 0.0, b1 = 0.0;
#pragma unroll
          for (int i = 0; i < 5; ++i) {
            dq2[i] = yq[i] - pt.oq[i];
            df2[i] = f[i] - pt.of[i];
            const double o = pt.odf[i];
            G22 += df2[i] * df2[i];
            b2 += df2[i] * f[i];
            G11o += o * o;
            G12 += o * df2[i];
            b1 += o * f[i];
          }
          double g1, g2;
          anderson2(omem == 3, G11o, G12, G22, b1, b2, g1, g2);
#pragma unroll
          for (int i = 0; i < 5; ++i) {
            yn[i] = yq[i] - g2 * dq2[i] - g1 * pt.odq[i];
            pt.odq[i] = dq2[i];
            pt.odf[i] = df2[i];
          }
        }
        bool finite = true;
#pragma unroll
        for (int i = 0; i < 5; ++i) {
          pt.oq[i] = yq[i];
          pt.of[i] = f[i];
          finite = finite && isfinite(yn[i]);
        }
        if (!finite) {
          status = NMC_STATUS_NONFINITE;
          fatal = true;
          run = false;
        } else {
          // Algorithm outerConverged: Ye and ef componentwise against y*,
          // each velocity component against the speed max(|v*|, |v^[k+1]|)
          const double vst = sqrt(pt.yst[2] * pt.yst[2] + pt.yst[3] * pt.yst[3] + pt.yst[4] * pt.yst[4]);
          const double vnw = sqrt(yn[2] * yn[2] + yn[3] * yn[3] + yn[4] * yn[4]);
          const double vref = vst > vnw ? vst : vnw;
          bool oc = fabs(yn[0] - pt.y[0]) <= a->prm.tol_outer * fabs(pt.yst[0]) &&
                    fabs(yn[1] - pt.y[1]) <= a->prm.tol_outer * fabs(pt.yst[1]);
#pragma unroll
          for (int j = 0; j < 3; ++j) oc = oc && fabs(yn[2 + j] - pt.y[2 + j]) <= a->prm.tol_outer * vref;
#pragma unroll
          for (int i = 0; i < 5; ++i) pt.y[i] = yn[i];
          if (oc) {
            outer_conv = true;
            run = false;
          }
        }
      }
    }
    if (!skip && !fatal) {
      if (!outer_conv) status = NMC_STATUS_MAX_OUTER;
      else if (inner_failed) status = NMC_STATUS_MAX_INNER;
    }

    // ---- outputs --------------------------------------------------------
    // matter right-hand side at the final moments and the matter iterate they
    // were solved at
    const_ptr<FwdVArgs> ao = kernel_args<FwdVArgs>();
    const_ptr<DevModel> mo = scalar_ptr(ao->mdl);
    double yout[5], T_out;
    {
      const double vu[3] = {pt.yused[2], pt.yused[3], pt.yused[4]};
      double X[5];
      eulerian(S, mo, sp, lane, q0, D, I, vu, X);
      matter_rhs(pt, K, X, yout);
    }
    if (skip || ao->prm.fixed_matter) {
#pragma unroll
      for (int i = 0; i < 5; ++i) yout[i] = pt.yst[i];
      T_out = T_last;
    } else {
      T_out = temperature(mo, yout, r3);
    }
    if (has_point) {
      in_global(ao->D)[oD] = D;
#pragma unroll
      for (int j = 0; j < 3; ++j) in_global(ao->I)[oI + j * NQ] = I[j];
      if (threadIdx.x == (h << 5)) {  // wave 0, first lane of the half
        in_global(ao->ye)[p] = yout[0];
        in_global(ao->ef)[p] = yout[1];
#pragma unroll
        for (int j = 0; j < 3; ++j) in_global(ao->v)[3 * p + j] = yout[2 + j];
        in_global(ao->T)[p] = T_out;
        in_global(ao->n_outer)[p] = skip ? 0 : k_done;
        in_global(ao->n_inner)[p] = total_inner;
        in_global(ao->status)[p] = status;
      }
    }
    __syncthreads();  // LDS is free for the next pair
  }
};

template <int NS, bool PHI1>
__global__ __launch_bounds__(kLanes* NS, 2) void fwd_vsplit_kernel(FwdVArgs a) {
  __shared__ VSplitLds<NS, PHI1> S;
  load_model(a.mdl, a.theta, S.m);
  const int64_t pairs = (a.P + 1) / 2;
  for (int64_t u = blockIdx.x; u < pairs; u += gridDim.x) VSplitSolver<NS, PHI1>::solve(u, S);
}

template <int NS, bool PHI1>
hipError_t launch_vsplit_t(const FwdVArgs& a, const nmc_launch& L, int num_cu, hipStream_t s) {
  hipLaunchKernelGGL((fwd_vsplit_kernel<NS, PHI1>), dim3((unsigned)split_grid(L, a.P, num_cu)), dim3(kLanes * NS), 0, s,
                     a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_forward_vsplit(const FwdVArgs& a, int ns, bool phi1, const nmc_launch& L, int num_cu, hipStream_t s) {
  if (ns == 2) return phi1 ? launch_vsplit_t<2, true>(a, L, num_cu, s) : launch_vsplit_t<2, false>(a, L, num_cu, s);
  if (ns == 3) return phi1 ? launch_vsplit_t<3, true>(a, L, num_cu, s) : launch_vsplit_t<3, false>(a, L, num_cu, s);
  return hipErrorInvalidValue;
}

}  // namespace nmc
