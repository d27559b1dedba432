// Forward kernel of the implicit coupling solve for 64 energy nodes (CDNA4).
//
// Same algorithm as the 32-node kernel (Algorithm neutrinoMatterCoupling,
// Sec. 3.5.3), different data placement.  The four 64 x 64 kernel matrices of
// a point (128 KiB) fit neither in one wavefront's registers nor, at useful
// occupancy, in LDS, so they are not stored at all.
//
// One 64-lane wavefront solves one point; lane q owns D_s[q] and I_s[q] of
// every species.  All four kernels share one symmetric core: with
// g = exp(-e / (2T)), h = g^2 and B2(q, j) = exp(-|e_q - e_j| / T),
//   Phi_in[q][j] = A e_q e_j B2 g_q / g_j,  Phi_out[q][j] = A e_q e_j B2 g_j / g_q,
//   Phi_ann = A' e_q e_j B2,                Phi_pro = A' e_q e_j B2 h_q h_j,
// and every inner iteration contracts B2 against W e D / g, g W e (1 - D),
// W e D and h W e (1 - D).  B2 is semiseparable: for q and j in different
// blocks of nodes, with b the node of j's block next to q's, B2(q, j) =
// B2(q, b) B2(b, j).  A lane keeps the 16 entries of its own 16-lane row (FMAs
// that take column j by DPP row_newbcast), one coefficient for the other row
// of its half and one for the other half, formed once per outer iteration; the
// sums at the neighbouring nodes arrive by one lane exchange each
// (ds_swizzle, ds_bpermute).  19 multiply-adds and two exchanges per vector
// instead of 64 and the vector's redistribution.  g and 1 / g are scaled by
// 2^+-c, c the middle of the point's exponent range.  Instruction issue at two
// waves per SIMD and, for small batches, the dependent reductions bound it:
// 131072 points of the radial profile take 1.69 ms (3.10 ms with rows of 64
// entries in registers, 4.84 ms with every column regenerated from LDS in
// every inner iteration), 1001 points 71 us (124 us, 233 us).
//
// Where the grid spans more than kDirectBits64 powers of two in g (T below
// ~0.22 MeV) the lanes instead regenerate their rows column by column in every
// inner iteration from per-node exponent splits broadcast from LDS (`rates`).
// With (lo, hi) the lower / higher node of the pair:
//   b = exp(-(e_hi - e_lo) / (2T)) = ldexp(P_lo R_hi, n_lo - n_hi),
//   Phi_in[q][j] = A e_q e_j (j > q ? b : b^3),  Phi_out[q][j] = A e_q e_j (j > q ? b^3 : b),
//   Phi_ann[q][j] = A' e_q e_j b^2,              Phi_pro[q][j] = A' e_q e_j G_hi,
// with x = e log2(e) / (2T) = n + f, P = 2^f, R = 2^-f, G = exp(-2 e / T):
// every factor at most 1.  Anderson sums, norms and matter integrals are
// full-wave register reductions.
//
// The PRE variant (kernel_store = HBM; the roofline study of precomputed
// kernels) writes the entries and coefficients to the workspace once per outer
// iteration, laid out [entry][lane] so that every access is a coalesced
// 512-byte wave load or store, and reads them back in every inner iteration.  Each lane
// reads only what it wrote, so no barrier is needed between the two.  Both
// variants perform the same floating-point operations on the same values, so
// their results agree bit for bit.
#include "nmc_pair.h"

namespace nmc {
namespace {

constexpr int NQ64 = 64;
// widest exponent range of g for the register rows: squares of the scaled
// factors and their reciprocals stay inside the normal range
constexpr int kDirectBits64 = 1000;
// per lane: the entries of its 16-lane row, the other row's coefficient, the
// other half's
constexpr int kCore = 18;

template <int NS>
struct Lds64 {
  ModelLdsN<NQ64> m;
  double hist[2][2 * NS][kLanes];  // Anderson history per owned moment: Q_prev, F_prev
  double colPR[kLanes][2];         // per node: P, R of the exponent split at the current T
  double colGE[kLanes][2];         // per node: G = exp(-2 e / T), W e
  int coln[kLanes];                // per node: integer part n of the split
  double X[NS][kLanes];            // W e D of the current iterate
  // uniform per-point state
  double dref[NS];
  double y[2], oq[2], of[2], odq[2], odf[2];
  double T_last, r3, K, An, Ap;
  // per-point inputs read in every outer iteration, staged once per point
  double ye_st, e_st, chi0, T_fix, mu_fix;
};

// sums over the wave of V <= 12 lane values, in every lane
template <int V>
__device__ __forceinline__ void wave_sums(const double (&v)[V], double (&out)[V]) {
  static_for<0, (V + 3) / 4>([&](auto cc) {
    constexpr int c = decltype(cc)::value;
    double in[4], o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) in[i] = (4 * c + i < V) ? v[(4 * c + i < V) ? 4 * c + i : 0] : 0.0;
    wave_sums4(in, o);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (4 * c + i < V) out[4 * c + i] = o[i];
  });
}

template <int NS, bool COUPLED, bool PRE>
struct PointSolver64 {
  static constexpr int NQ = NQ64;

  // entries of row q, column j of the four kernels without their common
  // factor A e_q e_j (A' e_q e_j for pair): e_j rides on the contracted
  // vectors and A e_q scales the row sums
  struct Row {
    double Pq, Rq, Gq;
    int nq;
  };
  __device__ __forceinline__ static Row row_consts(const Lds64<NS>& S, int q) {
    Row r;
    r.Pq = S.colPR[q][0];
    r.Rq = S.colPR[q][1];
    r.Gq = S.colGE[q][0];
    r.nq = S.coln[q];
    return r;
  }
  // per-node data of column j, read from LDS one column ahead of its use
  struct Col {
    double P, R, G, w, x[NS];
    int n;
  };
  __device__ __forceinline__ static Col load_col(const Lds64<NS>& S, int j) {
    Col c;
    c.P = S.colPR[j][0];
    c.R = S.colPR[j][1];
    c.G = S.colGE[j][0];
    c.w = S.colGE[j][1];
    c.n = S.coln[j];
#pragma unroll
    for (int t = 0; t < NS; ++t) c.x[t] = S.X[t][j];
    return c;
  }
  // u = 2^(x_q - x_j) and v = 2^(x_j - x_q): the one not above 1 is
  // b = exp(-|e_q - e_j| / (2T)), the other its reciprocal (or +inf), so
  // Phi_in = (j > q ? b : b^3) = min(u, v^3), Phi_out = min(u^3, v) and
  // Phi_ann = b^2 = min(u^2, v^2) without a compare or select
  __device__ __forceinline__ static void entries(const Col& c, const Row& r, double& fin, double& fout,
                                                 double& fann, double& fpro) {
    const int e = r.nq - c.n;
    const double u = ldexp(r.Pq * c.R, e), v = ldexp(c.P * r.Rq, -e);
    const double u2 = u * u, v2 = v * v;
    fin = min_f64(u, v2 * v);
    fout = min_f64(u2 * u, v);
    fann = min_f64(u2, v2);
    fpro = min_f64(c.G, r.Gq);  // G of the higher node: G falls with energy
  }
  __device__ __forceinline__ static void accumulate(const Col& c, double fin, double fout, double fann, double fpro,
                                                    double (&etaN)[NS], double (&outN)[NS], double (&annP)[NS],
                                                    double (&etaP)[NS]) {
    double x[NS], y[NS];
#pragma unroll
    for (int t = 0; t < NS; ++t) {
      x[t] = c.x[t];
      y[t] = c.w - x[t];
    }
#pragma unroll
    for (int t = 0; t < NS; ++t) {
      const int tb = pair_partner<NS>(t);
      etaN[t] = __builtin_fma(fin, x[t], etaN[t]);
      outN[t] = __builtin_fma(fout, y[t], outN[t]);
      annP[t] = __builtin_fma(fann, x[tb], annP[t]);
      etaP[t] = __builtin_fma(fpro, y[tb], etaP[t]);
    }
  }

  // The four contractions of every species at the current iterate, columns
  // regenerated from the splits in LDS (X holds W e D): etaN = Phi_in W D_s,
  // outN = Phi_out W (1 - D_s), annP = Phi_ann W D_sbar,
  // etaP = Phi_pro W (1 - D_sbar), without the factors A e_q of the row
  __device__ __forceinline__ static void rates(const Lds64<NS>& S, int q, double (&etaN)[NS], double (&outN)[NS],
                                               double (&annP)[NS], double (&etaP)[NS]) {
    const Row r = row_consts(S, q);
    auto column = [&](const Col& c) __attribute__((always_inline)) {
      double fin, fout, fann, fpro;
      entries(c, r, fin, fout, fann, fpro);
      accumulate(c, fin, fout, fann, fpro, etaN, outN, annP, etaP);
    };
    // two column buffers in turn: the reads of one overlap the work on the
    // other (the last trip re-reads column 0, unused)
    Col ca = load_col(S, 0), cb;
#pragma unroll 1
    for (int j = 0; j < NQ; j += 2) {
      cb = load_col(S, j + 1);
      column(ca);
      ca = load_col(S, (j + 2) & (NQ - 1));
      column(cb);
    }
  }

  // The four contractions of every species on the core: the lane's half as in
  // the 32-node kernels, then the other half's columns by the sum that its
  // node next to this half has (node 32 for the lower half, 31 for the upper)
  __device__ __forceinline__ static void contract(const double (&C)[kCore], const double (&a)[NS],
                                                  const double (&b)[NS], const double (&c)[NS], const double (&d)[NS],
                                                  double (&eN)[NS], double (&oN)[NS], double (&aP)[NS],
                                                  double (&eP)[NS]) {
    double B[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) B[j] = C[j];
    pairk::core_contract<NS>(B, C[16], a, b, c, d, eN, oN, aP, eP);
    const int from = (threadIdx.x & 32) ? 31 * 4 : 32 * 4;
    auto other = [&](double v) {
      return mk64((uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)lo32(v)),
                  (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)hi32(v)));
    };
    double z[4][NS];
#pragma unroll
    for (int t = 0; t < NS; ++t) {
      z[0][t] = other(eN[t]);
      z[1][t] = other(oN[t]);
      z[2][t] = other(aP[t]);
      z[3][t] = other(eP[t]);
    }
#pragma unroll
    for (int t = 0; t < NS; ++t) {
      eN[t] = __builtin_fma(C[17], z[0][t], eN[t]);
      oN[t] = __builtin_fma(C[17], z[1][t], oN[t]);
      aP[t] = __builtin_fma(C[17], z[2][t], aP[t]);
      eP[t] = __builtin_fma(C[17], z[3][t], eP[t]);
    }
  }

  // settle() is called once the point's inputs are loaded (work-queue hook)
  template <class Settle>
  __device__ __forceinline__ static void solve(int64_t p, Lds64<NS>& S, Settle&& settle) {
    const_ptr<FwdArgs> a = kernel_args<FwdArgs>();
    const_ptr<DevModel> md = scalar_ptr(a->mdl);
    const ModelLdsN<NQ>& mt = S.m;
    const int lane = threadIdx.x;
    const int q0 = lane;
    const double dtau = a->dtau;
    const int64_t base = p * (int64_t)(NS * NQ);
    const double rho = in_global(a->rho11)[p];
    const bool fixedT = a->prm.fixed_matter && a->T_fixed;
    // this lane's entries of the stored core
    double* __restrict__ kst = PRE ? a->kstore + p * (int64_t)(kCore * NQ) + lane : nullptr;

    double D[NS], I[NS];
#pragma unroll
    for (int t = 0; t < NS; ++t) {
      const int64_t o = base + md->ext[t] * NQ + lane;
      D[t] = in_global(a->D0)[o];
      I[t] = in_global(a->I0)[o];
    }
    // the old moments are read again where they are used (the outputs, which
    // may be the same arrays, are written at the end), so that they hold no
    // registers beside the row of the core
    auto old = [&](const double* x, int t, const_ptr<DevModel> m) {
      return in_global(x)[base + m->ext[t] * NQ + opaque(lane)];
    };

    settle();
    if (rho < md->rho11_min) {
      // coupling disabled at low density (Sec. 7.2): pass the state through
#pragma unroll
      for (int t = 0; t < NS; ++t) {
        const int64_t o = base + md->ext[t] * NQ + lane;
        in_global(a->D)[o] = D[t];
        in_global(a->I)[o] = I[t];
      }
      if (lane == 0) {
        const double ye_st = in_global(a->ye0)[p], e_st = in_global(a->e0)[p];
        in_global(a->ye)[p] = ye_st;
        in_global(a->e)[p] = e_st;
        in_global(a->T)[p] = fixedT ? in_global(a->T_fixed)[p]
                        : (e_st - md->eos_b * ye43(ye_st) * cbrt(rho)) / (md->eos_a * (1.0 + ye_st));
        in_global(a->n_outer)[p] = 0;
        in_global(a->n_inner)[p] = 0;
        in_global(a->status)[p] = NMC_STATUS_OK;
      }
      return;
    }

    S.r3 = cbrt(rho);
    S.K = md->kcoup / rho;
    S.An = (md->flags & NMC_NES) ? mt.theta[NQ] * rho : 0.0;
    S.Ap = (md->flags & NMC_PAIR) ? mt.theta[NQ + 1] * rho : 0.0;
    {
      const double w2q = mt.w2[q0];
      double v[NS], s[NS];
#pragma unroll
      for (int t = 0; t < NS; ++t) v[t] = w2q * D[t] * D[t];
      wave_sums<NS>(v, s);
#pragma unroll
      for (int t = 0; t < NS; ++t) S.dref[t] = s[t];
    }
    S.ye_st = S.y[0] = in_global(a->ye0)[p];
    S.e_st = S.y[1] = in_global(a->e0)[p];
    S.chi0 = a->chi0 ? in_global(a->chi0)[p] : md->chi_ref * rho;
    if (fixedT) S.T_fix = in_global(a->T_fixed)[p];
    if (a->prm.fixed_matter && a->mu_fixed) S.mu_fix = in_global(a->mu_fixed)[p];
#pragma unroll
    for (int i = 0; i < 2; ++i) S.oq[i] = S.of[i] = S.odq[i] = S.odf[i] = 0.0;
    S.T_last = 0.0;

    int status = NMC_STATUS_OK;
    bool fatal = false, inner_failed = false, outer_conv = false;
    int k, total_inner = 0;

    for (k = 1; k <= a->prm.max_outer; ++k) {
      // per-iteration opaque copies keep lane invariants from being hoisted
      // out of this loop (and spilled)
      const_ptr<FwdArgs> a = kernel_args<FwdArgs>();
      const_ptr<DevModel> md = scalar_ptr(a->mdl);
      const int q = opaque(q0);
      // ---- ComputeOpacities(y^[k]) --------------------------------------
      // (refined reciprocals as at 32 nodes: 131072 points 1732 -> 1689 us, 1001
      // points 72.2 -> 70.8 us; the series logarithm issues less but its chain is
      // longer: 1659 and 73.4 us)
      const double r3 = S.r3;
      const double y0 = S.y[0], y1 = S.y[1];
      const double T = fixedT ? S.T_fix : (y1 - md->eos_b * ye43(y0) * r3) * rcp_nr(md->eos_a * (1.0 + y0));
      const double mu = (a->prm.fixed_matter && a->mu_fixed)
                            ? S.mu_fix
                            : md->mu_a * (y0 - md->mu_ye0) * r3 + md->mu_b * log(T * md->inv_mu_t0);
      if (!(T > 0.0) || !(y0 >= 0.0) || !isfinite(T) || !isfinite(mu)) {
        status = NMC_STATUS_EOS_DOMAIN;
        fatal = true;
        break;
      }
      S.T_last = T;
      const double invT = rcp_nr(T);
      // constant parts of the numerator and denominators of Q (Eqs.
      // emissivityEmAbNodal, transportOpacityNodal, implicitMomentsNodal)
      double baseD[NS], den0D[NS];
      double dsig = 0.0;  // dtau sigma: 1 + dtau kappa = 1 + dtau chi + dsig
      const double epsq = mt.eps[q];
      {
        const double chi0 = S.chi0;
        const double shape = chi0 * mt.shape[q];
        const double sig = (md->flags & NMC_ISO) ? md->sigma_ratio * shape : 0.0;
        const double emab_q = (md->flags & NMC_EMAB) ? mt.theta[q] * shape : 0.0;
#pragma unroll
        for (int t = 0; t < NS; ++t) {
          const double chia = md->iemab[t] * emab_q;
          double deq = 0.0;
          if (!(NS == 3 && t == 2)) {
            // three species are nu_e, anti-nu_e, nu_x in this order, and nu_x
            // has no emission or absorption (chia = 0): no equilibrium
            const double x = (epsq - md->imusign[t] * mu) * invT;
            const double ex = exp(-fabs(x));
            const double r = rcp_nr(1.0 + ex);
            deq = x > 0.0 ? ex * r : r;
          }
          baseD[t] = old(a->D0, t, md) + dtau * (chia * deq);
          den0D[t] = 1.0 + dtau * chia;
        }
        dsig = dtau * sig;
      }
      // the lane's entries of the core and the node's factors, or the splits
      // in LDS
      double C[COUPLED && !PRE ? kCore : 1];
      double gq = 1.0, rgq = 1.0, hq = 1.0;
      bool direct = false;  // uniform
      if constexpr (COUPLED) {
        const ExpSplit xs = exp_split(epsq, invT);
        const int nlo = __builtin_amdgcn_readlane(xs.n, 0), nhi = __builtin_amdgcn_readlane(xs.n, NQ - 1);
        direct = nhi - nlo <= kDirectBits64;
        if (direct) {
          const int c = (nlo + nhi) >> 1;
          gq = ldexp(xs.R, c - xs.n);
          rgq = ldexp(xs.P, xs.n - c);
          hq = ldexp(xs.R * xs.R, -2 * xs.n);  // exp(-e / T)
          const double ht = gq * gq, rht = rgq * rgq;
          double B[16], kx;
          pairk::direct_row_regs(ht, rht, B, kx);
          const double up = readlane(ht, 32) * rht, down = ht * readlane(rht, 31);
          const double core[2] = {kx, (q & 32) ? down : up};
#pragma unroll
          for (int j = 0; j < kCore; ++j) {
            const double b = j < 16 ? B[j < 16 ? j : 0] : core[j < 16 ? 0 : j - 16];
            if constexpr (PRE) kst[j * NQ] = b;
            else C[j] = b;
          }
        } else {
          const double R2 = xs.R * xs.R;
          S.colPR[q][0] = xs.P;
          S.colPR[q][1] = xs.R;
          S.colGE[q][0] = ldexp(R2 * R2, -4 * xs.n);  // exp(-2 e / T)
          S.colGE[q][1] = mt.w2[q] * epsq;
          S.coln[q] = xs.n;
        }
      }

      // ---- inner loop over moments at fixed matter ------------------------
      const double w2q = mt.w2[q], w2eq = w2q * epsq;
      const double Aeq = S.An * epsq, Apq = S.Ap * epsq;
      double G11 = 0.0;
      double H[2][2 * NS];  // Anderson history: dQ_old, dF_old per owned moment (the previous Q and F in LDS)
      bool conv = false;
      const int m_inner = held(a->prm.m_inner), max_inner = held(a->prm.max_inner);
      const double tol2 = held(a->tol_inner2);
      const double* I0 = held(a->I0);
      int l;
      for (l = 1; l <= max_inner; ++l) {
        double etaN[NS], outN[NS], annP[NS], etaP[NS];
#pragma unroll
        for (int t = 0; t < NS; ++t) etaN[t] = outN[t] = annP[t] = etaP[t] = 0.0;
        if constexpr (COUPLED) {
          if (direct) {
            double c[kCore];
#pragma unroll
            for (int j = 0; j < kCore; ++j) {
              if constexpr (PRE) {
                c[j] = kst[j * NQ];
              } else {
                asm volatile("" : "+v"(C[j]));
                c[j] = C[j];
              }
            }
            double xg[NS], yg[NS], xv[NS], hy[NS];
#pragma unroll
            for (int t = 0; t < NS; ++t) {
              xv[t] = w2eq * D[t];
              const double yv = __builtin_fma(-w2eq, D[t], w2eq);
              xg[t] = xv[t] * rgq;
              yg[t] = yv * gq;
              hy[t] = hq * yv;
            }
            contract(c, xg, yg, xv, hy, etaN, outN, annP, etaP);
          } else {
#pragma unroll
            for (int t = 0; t < NS; ++t) S.X[t][q] = w2eq * D[t];
            __syncthreads();
            rates(S, q, etaN, outN, annP, etaP);
            __syncthreads();
          }
        }
        // Q and residual of both moments (owned entries x = (D_t, I_t))
        double Qx[2 * NS], Fx[2 * NS];
#pragma unroll
        for (int t = 0; t < NS; ++t) {
          const double eta = __builtin_fma(Aeq * gq, etaN[t], Apq * hq * etaP[t]);
          const double chi = __builtin_fma(Aeq * rgq, outN[t], __builtin_fma(Apq, annP[t], eta));
          // one reciprocal of the product of the two denominators serves both
          const double dD = __builtin_fma(dtau, chi, den0D[t]), dI = dD + dsig;
          const double r = rcp_nr(dD * dI);
          Qx[t] = __builtin_fma(dtau, eta, baseD[t]) * (r * dI);
          Qx[NS + t] = old(I0, t, md) * (r * dD);
          Fx[t] = Qx[t] - D[t];
          Fx[NS + t] = Qx[NS + t] - I[t];
        }
        // Anderson step over min(l, M_inner) residuals (difference form)
        const int mem = l < m_inner ? l : m_inner;
        double Xn[2 * NS];
        if (mem == 1) {
          // clear the older difference column (weighted zero at the second
          // iterate), so that no stale value enters that product
#pragma unroll
          for (int x = 0; x < 2 * NS; ++x) {
            Xn[x] = Qx[x];
            H[0][x] = 0.0;
            H[1][x] = 0.0;
          }
        } else {
          const double use1 = (mem == 3) ? 1.0 : 0.0;
          double dQ2[2 * NS], dF2[2 * NS];
          double v4[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
          for (int x = 0; x < 2 * NS; ++x) {
            dQ2[x] = Qx[x] - S.hist[0][x][lane];
            dF2[x] = Fx[x] - S.hist[1][x][lane];
            const double dF1 = use1 * H[1][x];
            v4[0] += dF1 * dF2[x];
            v4[1] += dF2[x] * dF2[x];
            v4[2] += dF1 * Fx[x];
            v4[3] += dF2[x] * Fx[x];
          }
          double gs[4];
          wave_sums4(v4, gs);
          const double G12 = gs[0], G22 = gs[1], b1 = gs[2], b2 = gs[3];
          double g1, g2;
          anderson2(mem == 3, G11, G12, G22, b1, b2, g1, g2);
#pragma unroll
          for (int x = 0; x < 2 * NS; ++x) {
            Xn[x] = Qx[x] - g2 * dQ2[x] - g1 * H[0][x];
            H[0][x] = dQ2[x];
            H[1][x] = dF2[x];
          }
          G11 = G22;
        }
#pragma unroll
        for (int x = 0; x < 2 * NS; ++x) {
          S.hist[0][x][lane] = Qx[x];
          S.hist[1][x][lane] = Fx[x];
        }
        bool bad = false;
#pragma unroll
        for (int x = 0; x < 2 * NS; ++x) bad |= !isfinite(Xn[x]);
        if (wave_any(bad)) {
          status = NMC_STATUS_NONFINITE;
          fatal = true;
          break;
        }
        // Algorithm innerConverged, compared squared; the sums are spread over
        // the wave (row c of 16 lanes holds species c, spread_conv_sums64) and
        // the point has converged when every lane passes
        {
          double vd[NS], vi[NS], vn[NS];
#pragma unroll
          for (int t = 0; t < NS; ++t) {
            const double dd = Xn[t] - D[t], di = Xn[NS + t] - I[t];
            vd[t] = w2q * dd * dd;
            vi[t] = w2q * di * di;
            vn[t] = w2q * Xn[t] * Xn[t];
          }
          double dm2, dn2;
          spread_conv_sums64<NS>(vd, vi, vn, dm2, dn2);
          const int cls = lane >> 4;
          const double d0 = cls < NS ? S.dref[cls < NS ? cls : 0] : 0.0;
          const double dref2 = d0 > dn2 ? d0 : dn2;
          conv = __builtin_amdgcn_ballot_w64(!(dm2 <= tol2 * dref2)) == 0;
          if (conv && cls < NS) S.dref[cls < NS ? cls : 0] = dn2;
        }
#pragma unroll
        for (int t = 0; t < NS; ++t) {
          D[t] = Xn[t];
          I[t] = Xn[NS + t];
        }
        if (conv) break;
      }
      total_inner += (l > max_inner ? max_inner : l);
      if (fatal) break;
      if (!conv) {
        inner_failed = true;
        double v[NS], s[NS];
#pragma unroll
        for (int t = 0; t < NS; ++t) v[t] = w2q * D[t] * D[t];
        wave_sums<NS>(v, s);
#pragma unroll
        for (int t = 0; t < NS; ++t) S.dref[t] = s[t];
      }
      if (a->prm.fixed_matter) {
        outer_conv = true;
        break;
      }

      // ---- matter right-hand side (Eq. implicitFluidNodal at v = 0) -------
      double yq0, yq1;
      {
        const double w3 = mt.w3[q];
        double mv[2] = {0.0, 0.0}, s[2];
#pragma unroll
        for (int t = 0; t < NS; ++t) {
          const double dd = D[t] - old(a->D0, t, md);
          mv[0] += md->ig[t] * w2q * dd;
          mv[1] += md->imult[t] * w3 * dd;
        }
        wave_sums<2>(mv, s);
        yq0 = S.ye_st - S.K * s[0];
        yq1 = S.e_st - S.K * s[1];
      }
      const double f0 = yq0 - S.y[0], f1 = yq1 - S.y[1];
      const int omem = k < a->prm.m_outer ? k : a->prm.m_outer;
      double yn0, yn1;
      if (omem == 1) {
        yn0 = yq0;
        yn1 = yq1;
      } else {
        const double dq20 = yq0 - S.oq[0], dq21 = yq1 - S.oq[1];
        const double df20 = f0 - S.of[0], df21 = f1 - S.of[1];
        const double odf0 = S.odf[0], odf1 = S.odf[1];
        const double G22 = df20 * df20 + df21 * df21, b2 = df20 * f0 + df21 * f1;
        const double G11o = odf0 * odf0 + odf1 * odf1;
        const double G12 = odf0 * df20 + odf1 * df21, b1 = odf0 * f0 + odf1 * f1;
        double g1, g2;
        anderson2(omem == 3, G11o, G12, G22, b1, b2, g1, g2);
        yn0 = yq0 - g2 * dq20 - g1 * S.odq[0];
        yn1 = yq1 - g2 * dq21 - g1 * S.odq[1];
        S.odq[0] = dq20;
        S.odq[1] = dq21;
        S.odf[0] = df20;
        S.odf[1] = df21;
      }
      S.oq[0] = yq0;
      S.oq[1] = yq1;
      S.of[0] = f0;
      S.of[1] = f1;
      if (!isfinite(yn0) || !isfinite(yn1)) {
        status = NMC_STATUS_NONFINITE;
        fatal = true;
        break;
      }
      const bool oc = fabs(yn0 - S.y[0]) <= a->prm.tol_outer * fabs(S.ye_st) &&
                      fabs(yn1 - S.y[1]) <= a->prm.tol_outer * fabs(S.e_st);
      S.y[0] = yn0;
      S.y[1] = yn1;
      if (oc) {
        outer_conv = true;
        break;
      }
    }
    if (k > a->prm.max_outer) k = a->prm.max_outer;
    if (!fatal) {
      if (!outer_conv) status = NMC_STATUS_MAX_OUTER;
      else if (inner_failed) status = NMC_STATUS_MAX_INNER;
    }

    // ---- outputs --------------------------------------------------------
    const_ptr<FwdArgs> ao = kernel_args<FwdArgs>();
    const_ptr<DevModel> mo = scalar_ptr(ao->mdl);
    const double ye_st = S.ye_st, e_st = S.e_st;
    double ye_out = ye_st, e_out = e_st, T_out = S.T_last;
    if (!ao->prm.fixed_matter) {
      const double w2 = mt.w2[q0], w3 = mt.w3[q0];
      double mv[2] = {0.0, 0.0}, s[2];
#pragma unroll
      for (int t = 0; t < NS; ++t) {
        const double dd = D[t] - old(ao->D0, t, mo);
        mv[0] += mo->ig[t] * w2 * dd;
        mv[1] += mo->imult[t] * w3 * dd;
      }
      wave_sums<2>(mv, s);
      ye_out = ye_st - S.K * s[0];
      e_out = e_st - S.K * s[1];
      T_out = (e_out - mo->eos_b * ye43(ye_out) * S.r3) / (mo->eos_a * (1.0 + ye_out));
    } else if (status == NMC_STATUS_EOS_DOMAIN) {
      T_out = fixedT ? S.T_fix : (e_st - mo->eos_b * ye43(ye_st) * S.r3) / (mo->eos_a * (1.0 + ye_st));
    }
#pragma unroll
    for (int t = 0; t < NS; ++t) {
      const int64_t o = base + mo->ext[t] * NQ + lane;
      in_global(ao->D)[o] = D[t];
      in_global(ao->I)[o] = I[t];
    }
    if (lane == 0) {
      in_global(ao->ye)[p] = ye_out;
      in_global(ao->e)[p] = e_out;
      in_global(ao->T)[p] = T_out;
      in_global(ao->n_outer)[p] = k;
      in_global(ao->n_inner)[p] = total_inner;
      in_global(ao->status)[p] = status;
    }
    __syncthreads();
  }
};

template <int NS, bool COUPLED, bool PRE, bool QUEUE>
__global__ __launch_bounds__(kLanes, 2) void fwd64_kernel(FwdArgs a) {
  __shared__ Lds64<NS> S;
  load_model(a.mdl, a.theta, S.m);
  if constexpr (QUEUE) {
    WorkQueue wq(a.queue, a.P, a.chunk);
    for (int64_t g; (g = wq.next()) >= 0;) {
      const int64_t b0 = uniform64(g * a.chunk);
      const int64_t end = uniform64(b0 + a.chunk < a.P ? b0 + a.chunk : a.P);
      for (int64_t p = b0; p < end; ++p) PointSolver64<NS, COUPLED, PRE>::solve(p, S, [&] { wq.settle(); });
    }
  } else {
    const int64_t b0 = (int64_t)blockIdx.x * a.chunk;
    const int64_t end = b0 + a.chunk < a.P ? b0 + a.chunk : a.P;
    for (int64_t p = b0; p < end; ++p) PointSolver64<NS, COUPLED, PRE>::solve(p, S, [] {});
  }
}

template <int NS, bool COUPLED, bool PRE>
hipError_t launch64_t(FwdArgs a, const nmc_launch& L, int num_cu, hipStream_t s) {
  const LaunchPlan lp = plan_launch(L, a.P, 8, num_cu);
  a.chunk = lp.chunk;
  auto kern = fwd64_kernel<NS, COUPLED, PRE, false>;
  if (lp.queue) {
    const hipError_t e = launch_reset_counter(a.queue, s);
    if (e != hipSuccess) return e;
    kern = fwd64_kernel<NS, COUPLED, PRE, true>;
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)lp.grid), dim3(kLanes), 0, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_forward64(const FwdArgs& a, int ns, bool coupled, const nmc_launch& L, int num_cu,
                            hipStream_t s) {
  if (a.kstore) {
    if (!coupled) return hipErrorInvalidValue;
    switch (ns) {
      case 1: return launch64_t<1, true, true>(a, L, num_cu, s);
      case 2: return launch64_t<2, true, true>(a, L, num_cu, s);
      case 3: return launch64_t<3, true, true>(a, L, num_cu, s);
    }
  } else if (coupled) {
    switch (ns) {
      case 1: return launch64_t<1, true, false>(a, L, num_cu, s);
      case 2: return launch64_t<2, true, false>(a, L, num_cu, s);
      case 3: return launch64_t<3, true, false>(a, L, num_cu, s);
    }
  } else {
    switch (ns) {
      case 1: return launch64_t<1, false, false>(a, L, num_cu, s);
      case 2: return launch64_t<2, false, false>(a, L, num_cu, s);
      case 3: return launch64_t<3, false, false>(a, L, num_cu, s);
    }
  }
  return hipErrorInvalidValue;
}

}  // namespace nmc
