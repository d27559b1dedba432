// Forward kernel of the implicit coupling solve for 32 energy nodes and small
// batches: one work-group per pair of points, one wavefront per species
// (CDNA4).
//
// A batch that does not fill the chip takes as long as its slowest point, and
// in the two-points-per-wavefront kernel an inner iteration is ~690
// instructions of one wave: 216 multiply-adds of the rates, the Anderson step
// and the convergence sums of all species one after the other.  Here wave t of
// the work-group holds species t of both points (lane 32 h + q: node q of the
// point of half h) and does that species' share of all of it, ~340
// instructions; the waves of a work-group run on different SIMDs.  What
// depends on every species goes through LDS: the residuals (whose Gram sums the
// Anderson step needs), the number moments of the pair partner (contracted into
// this species' rates) and the convergence flags in every inner iteration (two
// barriers), the changes that the matter right-hand side sums in every outer
// one.  Everything that follows from them (Gram sums, EOS, Anderson
// coefficients, matter iterate, convergence) is computed by every wave from the
// same values with the same instructions, so the waves take every branch
// together.
//
// Same algorithm, status rules and skip rule as the two-point kernel, and the
// same bits: every sum over species adds the lane's terms in that kernel's
// order before the lanes are summed, and the sums of one species take its
// reduction tree.  So a point's result does not depend on the size of its
// batch.
#include "nmc_fdproj.h"
#include "nmc_split.h"

namespace nmc {
namespace {

using namespace pairk;
using namespace splitk;

template <int NS>
struct SplitLds {
  ModelLds m;
  SplitExp E[2];             // per point: exponent splits (points too cold for scaled factors)
  double D[NS][kLanes];      // next number moments of every species
  double odds[NS][kLanes];   // projected equilibrium: o = D / (1 - D)
  alignas(16) double F[NS][kLanes][2];  // residuals of the moments of every species
  double dd[NS][kLanes];     // change of the number moments since the old state
  int flag[NS][2];           // 1: converged, 2: a non-finite iterate
};

template <int NS, bool PROJ>
struct SplitSolver {
  static constexpr int NQ = NQP;

  // the lane's terms of the matter right-hand side, added over the species in
  // the two-point kernel's order, summed over the half
  __device__ __forceinline__ static void matter_sums(SplitLds<NS>& S, const_ptr<DevModel> md, int sp, int lane,
                                                     double w2, double w3, double dd, double (&m)[2]) {
    __syncthreads();  // the last changes have been read
    S.dd[sp][lane] = dd;
    __syncthreads();
    double v[2] = {0.0, 0.0};
#pragma unroll
    for (int t = 0; t < NS; ++t) {
      const double d = S.dd[t][lane];
      v[0] += md->ig[t] * w2 * d;
      v[1] += md->imult[t] * w3 * d;
    }
    half_own_sums<1>(v, m);
  }

  __device__ __forceinline__ static void solve(int64_t u, SplitLds<NS>& S) {
    const_ptr<FwdArgs> a = kernel_args<FwdArgs>();
    const_ptr<DevModel> md = scalar_ptr(a->mdl);
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
    const int64_t o = p * (int64_t)(NS * NQ) + md->ext[sp] * NQ + q0;
    const double rho = in_global(a->rho11)[p];
    const bool fixedT = a->prm.fixed_matter && a->T_fixed;
    const bool fixed_mu = a->prm.fixed_matter && a->mu_fixed;
    const double Dst = in_global(a->D0)[o], Ist = in_global(a->I0)[o];
    const double ye_st = in_global(a->ye0)[p], e_st = in_global(a->e0)[p];
    const double chi0 = a->chi0 ? in_global(a->chi0)[p] : md->chi_ref * rho;
    const double T_fix = fixedT ? in_global(a->T_fixed)[p] : 0.0;
    const double mu_fix = fixed_mu ? in_global(a->mu_fixed)[p] : 0.0;
    double D = Dst, I = Ist;
    S.D[sp][lane] = D;

    // coupling disabled at low density (Sec. 7.2): the state passes through
    const bool skip = rho < md->rho11_min;
    const double r3 = cbrt(rho), K = md->kcoup / rho;
    const double An = (md->flags & NMC_NES) ? mt.theta[NQ] * rho : 0.0;
    const double Ap = (md->flags & NMC_PAIR) ? mt.theta[NQ + 1] * rho : 0.0;
    double y0 = ye_st, y1 = e_st;
    double oq0 = 0.0, oq1 = 0.0, of0 = 0.0, of1 = 0.0, odq0 = 0.0, odq1 = 0.0, odf0 = 0.0, odf1 = 0.0;
    // ||D^[k,1]||_W^2 of this species
    auto norm = [&](double w2) {
      const double v[2] = {w2 * D * D, 0.0};
      double s[2];
      half_own_sums<1>(v, s);
      return s[0];
    };
    double dref = norm(mt.w2[q0]);
    __syncthreads();
    double Dp = S.D[pa][lane];  // number moment of the partner
    __syncthreads();

    int status = NMC_STATUS_OK;
    bool fatal = false, inner_failed = false, outer_conv = false;
    bool run = !skip;  // this half's point is still iterating the outer loop
    int k_done = 0, total_inner = 0;
    double T_last = 0.0;  // temperature of the last outer iteration this half ran

    for (int k = 1; k <= a->prm.max_outer && __builtin_amdgcn_ballot_w64(run) != 0; ++k) {
      const_ptr<FwdArgs> a = kernel_args<FwdArgs>();
      const_ptr<DevModel> md = scalar_ptr(a->mdl);
      const int q = opaque(q0);
      if (run) k_done = k;
      // ---- ComputeOpacities(y^[k]) --------------------------------------
      const double T = fixedT ? T_fix : (y1 - md->eos_b * ye43(y0) * r3) * rcp_nr(md->eos_a * (1.0 + y0));
      const double mu =
          fixed_mu ? mu_fix : md->mu_a * (y0 - md->mu_ye0) * r3 + md->mu_b * log_pos(T * md->inv_mu_t0);
      if (run && (!(T > 0.0) || !(y0 >= 0.0) || !isfinite(T) || !isfinite(mu))) {
        status = NMC_STATUS_EOS_DOMAIN;
        fatal = true;
        run = false;
      }
      T_last = run ? T : T_last;
      // a finished half keeps a harmless temperature
      const double Tu = run ? T : 1.0, muu = run ? mu : 0.0;
      const double invT = rcp_nr(Tu);
      const double epsq = mt.eps[q];
      const ExpSplit xs = exp_split(epsq, invT);
      const double shape = chi0 * mt.shape[q];
      const double dsig = dtau * ((md->flags & NMC_ISO) ? md->sigma_ratio * shape : 0.0);
      const double chia = md->iemab[sp] * ((md->flags & NMC_EMAB) ? mt.theta[q] * shape : 0.0);
      // equilibrium, and the detailed-balance factors of this species and
      // (h only) its partner
      double deq, go = 1.0, rgo = 1.0, ho = 1.0, hp = 1.0;
      if constexpr (PROJ) {
        double pD, pC;
        fdp::projected_node(a->mdl, q, Tu, md->imusign[sp] * muu, pD, pC);
        deq = pD;
        ho = pD / pC;
        rgo = 1.0 / sqrt(ho);
        go = ho * rgo;
        S.odds[sp][lane] = ho;
      } else {
        const double x = (epsq - md->imusign[sp] * muu) * invT;
        const double ex = exp(-fabs(x));
        const double r = rcp_nr(1.0 + ex);
        deq = x > 0.0 ? ex * r : r;
      }
      const double baseD = Dst + dtau * (chia * deq);
      const double den0D = 1.0 + dtau * chia;

      // row of the symmetric core with the nodes' factors g and 1 / g scaled
      // by 2^+-c (every wave of the work-group forms the same row), where the
      // grid spans at most kDirectBits powers of two; else from the exponent
      // splits in LDS (cold_rows), signed beyond kSymBits: the forms and the
      // lines between them are the two-point kernel's
      double B[16], kx;
      const double hq = ldexp(xs.R * xs.R, -2 * xs.n);  // exp(-e / T)
      const int lo0 = __builtin_amdgcn_readlane(xs.n, 0), hi0 = __builtin_amdgcn_readlane(xs.n, 31);
      const int lo1 = __builtin_amdgcn_readlane(xs.n, 32), hi1 = __builtin_amdgcn_readlane(xs.n, 63);
      const int nlo = h ? lo1 : lo0, nhi = h ? hi1 : hi0;
      const int c = (nlo + nhi) >> 1;
      const bool direct = __builtin_amdgcn_ballot_w64(run && nhi - nlo > kDirectBits) == 0;
      const bool sym = PROJ || __builtin_amdgcn_ballot_w64(run && nhi - nlo > kSymBits) == 0;
      const double gt = ldexp(xs.R, c - xs.n), rgt = ldexp(xs.P, xs.n - c);
      if constexpr (!PROJ) {
        go = sym ? gt : 1.0;
        rgo = sym ? rgt : 1.0;
      }
      if (direct) {
        direct_row_regs(gt * gt, rgt * rgt, B, kx);
        if constexpr (PROJ) __syncthreads();
      } else if (sym) {
        cold_rows<true>(S.E[h], q, xs, B, kx);
      } else {
        cold_rows<false>(S.E[h], q, xs, B, kx);
      }
      if constexpr (PROJ) hp = S.odds[pa][lane];
      else ho = hp = hq;

      // ---- inner loop over moments at fixed matter ------------------------
      const double w2q = mt.w2[q], w2eq = w2q * epsq;
      const double Aeq = An * epsq, Apq = Ap * epsq;
      const double ag = Aeq * go, arg = Aeq * rgo, aph = Apq * ho;
      double G11 = 0.0;
      // Anderson history: Q of this species, residuals of every species
      double Qp[2] = {0.0, 0.0}, dQo[2] = {0.0, 0.0}, Fp[2 * NS], dFo[2 * NS];
#pragma unroll
      for (int x = 0; x < 2 * NS; ++x) Fp[x] = dFo[x] = 0.0;
      const double dref0 = dref;
      const bool ran = run;  // this half runs this outer iteration
      bool act = run;        // this half is still iterating the inner loop
      bool cvd = false;      // this half's inner loop converged
      int l_done = 0;
      const int m_inner = held(a->prm.m_inner), max_inner = held(a->prm.max_inner);
      const double tol2 = held(a->tol_inner2);
      for (int l = 1; l <= max_inner && __builtin_amdgcn_ballot_w64(act) != 0; ++l) {
        if (act) l_done = l;
#pragma unroll
        for (int j = 0; j < 16; ++j) asm volatile("" : "+v"(B[j]));
        const double xv = w2eq * D, yv = w2eq - xv;
        double eN[1], oN[1], aP[1], eP[1];
        const double xp[1] = {w2eq * Dp}, hyp[1] = {hp * (w2eq - xp[0])};
        if (sym) {
          const double xg[1] = {xv * rgo}, yg[1] = {yv * go};
          core_contract<1>(B, kx, xg, yg, xp, hyp, eN, oN, aP, eP);
        } else {
          signed_split(B, kx, xv, yv, xp[0], hyp[0], eN[0], oN[0], aP[0], eP[0]);
        }
        // Q and residual of both owned moments; one reciprocal of the product
        // of the two denominators serves both
        double Q[2], Xn[2];
        {
          const double eta = __builtin_fma(ag, eN[0], aph * eP[0]);
          const double chi = __builtin_fma(arg, oN[0], __builtin_fma(Apq, aP[0], eta));
          const double dD = __builtin_fma(dtau, chi, den0D), dI = dD + dsig;
          const double r = rcp_nr(dD * dI);
          Q[0] = __builtin_fma(dtau, eta, baseD) * (r * dI);
          Q[1] = Ist * (r * dD);
          S.F[sp][lane][0] = Q[0] - D;
          S.F[sp][lane][1] = Q[1] - I;
        }
        __syncthreads();  // and the flags and moments of the last iterate have been read
        double F[2 * NS];  // in the two-point kernel's order: D of every species, then I
#pragma unroll
        for (int t = 0; t < NS; ++t) {
          F[t] = S.F[t][lane][0];
          F[NS + t] = S.F[t][lane][1];
        }
        // Anderson step over min(l, M_inner) residuals (difference form)
        const int mem = l < m_inner ? l : m_inner;
        if (mem == 1) {
          Xn[0] = Q[0];
          Xn[1] = Q[1];
          dQo[0] = dQo[1] = 0.0;
#pragma unroll
          for (int x = 0; x < 2 * NS; ++x) dFo[x] = 0.0;
        } else {
          double v4[4] = {0.0, 0.0, 0.0, 0.0}, gs[4];
#pragma unroll
          for (int x = 0; x < 2 * NS; ++x) {
            const double dF2 = F[x] - Fp[x];
            v4[0] += dFo[x] * dF2;
            v4[1] += dF2 * dF2;
            v4[2] += dFo[x] * F[x];
            v4[3] += dF2 * F[x];
            dFo[x] = dF2;
          }
          half_sums4(v4, gs);
          double g1, g2;
          anderson2(mem == 3, G11, gs[0], gs[1], gs[2], gs[3], g1, g2);
#pragma unroll
          for (int x = 0; x < 2; ++x) {
            const double dQ2 = Q[x] - Qp[x];
            Xn[x] = Q[x] - g2 * dQ2 - g1 * dQo[x];
            dQo[x] = dQ2;
          }
          G11 = gs[1];
        }
        Qp[0] = Q[0];
        Qp[1] = Q[1];
#pragma unroll
        for (int x = 0; x < 2 * NS; ++x) Fp[x] = F[x];
        // Algorithm innerConverged for this species (reference guarded by the
        // new norm, compared squared), and whether an iterate is non-finite
        const bool bad = half_any(!isfinite(Xn[0]) || !isfinite(Xn[1]), h);
        const double dd = Xn[0] - D, di = Xn[1] - I;
        const double vm[2] = {w2q * dd * dd, w2q * di * di};
        double dm2, dn2;
        conv_sums(vm, w2q * Xn[0] * Xn[0], dm2, dn2);
        const bool conv1 = !half_any(!(dm2 <= tol2 * (dref0 > dn2 ? dref0 : dn2)), h);
        if (q0 == 0) S.flag[sp][h] = (conv1 ? 1 : 0) | (bad ? 2 : 0);
        S.D[sp][lane] = Xn[0];
        __syncthreads();
        int all = 1, any = 0;
#pragma unroll
        for (int t = 0; t < NS; ++t) {
          all &= S.flag[t][h];
          any |= S.flag[t][h];
        }
        const double Dpn = S.D[pa][lane];
        if ((any & 2) && act) {
          status = NMC_STATUS_NONFINITE;
          fatal = true;
          act = run = false;
        }
        if (act) {
          D = Xn[0];
          I = Xn[1];
          Dp = Dpn;
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
      // matter right-hand side (Eq. implicitFluidNodal at v = 0), and the norm
      // of the current moments where a running point's inner loop failed
      if (__builtin_amdgcn_ballot_w64(run && !cvd) != 0) {
        const double n = norm(w2q);
        dref = (run && !cvd) ? n : dref;
      }
      double m[2];
      matter_sums(S, md, sp, lane, w2q, mt.w3[q], D - Dst, m);
      const double yq0 = ye_st - K * m[0], yq1 = e_st - K * m[1];
      if (a->prm.fixed_matter) {
        if (run) outer_conv = true;
        run = false;
      }
      if (run) {
        const double f0 = yq0 - y0, f1 = yq1 - y1;
        const int omem = k < a->prm.m_outer ? k : a->prm.m_outer;
        double yn0, yn1;
        if (omem == 1) {
          yn0 = yq0;
          yn1 = yq1;
        } else {
          const double dq20 = yq0 - oq0, dq21 = yq1 - oq1;
          const double df20 = f0 - of0, df21 = f1 - of1;
          const double G22 = df20 * df20 + df21 * df21, b2 = df20 * f0 + df21 * f1;
          const double G11o = odf0 * odf0 + odf1 * odf1;
          const double G12 = odf0 * df20 + odf1 * df21, b1 = odf0 * f0 + odf1 * f1;
          double g1, g2;
          anderson2(omem == 3, G11o, G12, G22, b1, b2, g1, g2);
          yn0 = yq0 - g2 * dq20 - g1 * odq0;
          yn1 = yq1 - g2 * dq21 - g1 * odq1;
          odq0 = dq20;
          odq1 = dq21;
          odf0 = df20;
          odf1 = df21;
        }
        oq0 = yq0;
        oq1 = yq1;
        of0 = f0;
        of1 = f1;
        if (!isfinite(yn0) || !isfinite(yn1)) {
          status = NMC_STATUS_NONFINITE;
          fatal = true;
          run = false;
        } else {
          // Algorithm outerConverged: componentwise against y*
          const bool oc =
              fabs(yn0 - y0) <= a->prm.tol_outer * fabs(ye_st) && fabs(yn1 - y1) <= a->prm.tol_outer * fabs(e_st);
          y0 = yn0;
          y1 = yn1;
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
    const_ptr<FwdArgs> ao = kernel_args<FwdArgs>();
    const_ptr<DevModel> mo = scalar_ptr(ao->mdl);
    double ye_out = ye_st, e_out = e_st, T_out = T_last;
    {
      // the matter right-hand side at the final moments
      double m[2];
      matter_sums(S, mo, sp, lane, mt.w2[q0], mt.w3[q0], D - Dst, m);
      if (!skip && !ao->prm.fixed_matter) {
        ye_out = ye_st - K * m[0];
        e_out = e_st - K * m[1];
      }
      if (skip || !ao->prm.fixed_matter || status == NMC_STATUS_EOS_DOMAIN)
        T_out = fixedT ? T_fix : (e_out - mo->eos_b * ye43(ye_out) * r3) / (mo->eos_a * (1.0 + ye_out));
    }
    if (has_point) {
      in_global(ao->D)[o] = D;
      in_global(ao->I)[o] = I;
      if (threadIdx.x == (h << 5)) {  // wave 0, first lane of the half
        in_global(ao->ye)[p] = ye_out;
        in_global(ao->e)[p] = e_out;
        in_global(ao->T)[p] = T_out;
        in_global(ao->n_outer)[p] = skip ? 0 : k_done;
        in_global(ao->n_inner)[p] = total_inner;
        in_global(ao->status)[p] = status;
      }
    }
    __syncthreads();  // LDS is free for the next pair
  }
};

template <int NS, bool PROJ>
__global__ __launch_bounds__(kLanes* NS, 2) void fwd_split_kernel(FwdArgs a) {
  __shared__ SplitLds<NS> S;
  load_model(a.mdl, a.theta, S.m);
  const int64_t pairs = (a.P + 1) / 2;
  for (int64_t u = blockIdx.x; u < pairs; u += gridDim.x) SplitSolver<NS, PROJ>::solve(u, S);
}

template <int NS, bool PROJ>
hipError_t launch_split_t(const FwdArgs& a, const nmc_launch& L, int num_cu, hipStream_t s) {
  hipLaunchKernelGGL((fwd_split_kernel<NS, PROJ>), dim3((unsigned)split_grid(L, a.P, num_cu)), dim3(kLanes * NS), 0, s,
                     a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_forward_split(const FwdArgs& a, int ns, bool proj, const nmc_launch& L, int num_cu, hipStream_t s) {
  if (ns == 2) return proj ? launch_split_t<2, true>(a, L, num_cu, s) : launch_split_t<2, false>(a, L, num_cu, s);
  if (ns == 3) return proj ? launch_split_t<3, true>(a, L, num_cu, s) : launch_split_t<3, false>(a, L, num_cu, s);
  return hipErrorInvalidValue;
}

}  // namespace nmc
