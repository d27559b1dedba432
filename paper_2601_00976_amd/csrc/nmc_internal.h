// Internal declarations of the nmc library (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/nmc.h"

namespace nmc {

constexpr int kMaxNq = 64;
constexpr int kMaxNs = 3;
constexpr int kAdjPartials = 4096;  // most work-groups of either adjoint kernel, a row of partial sums each

// Model table resident in device memory.  The kernels copy the per-node
// tables into LDS once per work-group and read the uniform scalars through
// the scalar cache.
struct DevModel {
  int ns, nq;
  unsigned flags;
  int pad0;
  int species[kMaxNs];
  int partner[kMaxNs];  // index of the pair partner in the species list, or -1
  double g[kMaxNs];       // lepton number of the species
  double mult[kMaxNs];    // energy multiplicity (4 for the heavy-lepton stand-in)
  double musign[kMaxNs];  // chemical potential = musign * mu_nu_e
  double emab[kMaxNs];    // 1 if the species has emission/absorption
  // Internal species order used by the solve kernels: sorted by species id,
  // so that pair partners sit at compile-time positions (nu_e, anti-nu_e at
  // 0, 1 and nu_x last).  ext[t] is the caller's slot of internal species t;
  // the i* arrays are the per-species constants in internal order.
  int ext[kMaxNs];
  double ig[kMaxNs], imult[kMaxNs], imusign[kMaxNs], iemab[kMaxNs];
  double eps[kMaxNq];     // node energies [MeV]
  double w2[kMaxNq];      // w eps^2 dEps [MeV^3]
  double w3[kMaxNq];      // w2 eps [MeV^4]
  double shape[kMaxNq];   // (eps / eps_ref)^chi_power
  double chi_ref, sigma_ratio;
  double eos_a, eos_b, mu_a, mu_ye0, mu_b, mu_t0;
  double inv_mu_t0;       // 1 / mu_t0
  double kcoup;           // K * rho11 [MeV^-3]
  double rho11_min;
  double phi1_nes, phi1_pair;  // Phi_1 / Phi_0 of the NES and pair kernels
  // projected equilibrium (Eq. fermiDiracProjection) with its limiter bounds
  // D_min and 1 - D_max, and per-node tables of the node's element: edges,
  // l_1 eps^2 = pl[0] eps^3 + pl[1] eps^2 and l_2 likewise (pl[2], pl[3]),
  // the node's row of the inverse eps^2 mass matrix, 1 / int eps^2, and the
  // node's own basis function at the element's lower and upper edge
  int fd_projection;
  double deq_min, ceq_min;
  double pelo[kMaxNq], pehi[kMaxNq];
  double pl[kMaxNq][4];
  double pinv[kMaxNq][2];
  double prm0[kMaxNq];
  double pedge[kMaxNq][2];
};

struct SolverParams {
  double tol_inner, tol_outer;
  int m_inner, m_outer, max_inner, max_outer, fixed_matter;
};

struct FwdArgs {
  const DevModel* mdl;
  SolverParams prm;
  double tol_inner2;  // tol_inner^2 (the inner test is evaluated squared)
  int64_t P;
  double dtau;
  const double *D0, *I0, *rho11, *ye0, *e0, *chi0, *T_fixed, *mu_fixed, *theta;
  double *D, *I, *ye, *e, *T;
  int32_t *n_outer, *n_inner, *status;
  double* kstore;  // per-point kernel matrices (kernel_store = HBM) or nullptr
  int* queue;  // work-queue counters (persistent mode) or nullptr
  int chunk;   // units per grab
};

// O(v) forward solve (nonzero fluid velocity): moments D (P, ns, nq) and I
// (P, ns, 3, nq), matter (Ye, ef, v) with v (P, 3)
struct FwdVArgs {
  const DevModel* mdl;
  SolverParams prm;
  double tol_inner2;
  int64_t P;
  double dtau;
  const double *D0, *I0, *rho11, *ye0, *ef0, *v0, *chi0, *theta;
  double *D, *I, *ye, *ef, *v, *T;
  int32_t *n_outer, *n_inner, *status;
  int* queue;
  int chunk;
};

// the stage-3 input of a PD-ARS step (see nmc_primitive.hip)
struct PdarsArgs {
  int64_t P;
  int ns, nq;
  double w;          // a_32 / a_22: weight of stage 2 in U^(3*)
  double rho11_min;  // coupling density
  const double *rho11, *D0, *I0, *ye0, *ef0, *v0;  // the step's initial state
  const double *D2, *I2, *ye2, *ef2, *v2;          // stage-2 solution
  double *D3, *I3, *ye3, *ef3, *v3;                // stage-3 initial state
  int32_t* iters;    // recovery iterations per (point, species, node)
  int mem, max_it;   // recovery: Anderson memory and cap
  double tol2;       // recovery: squared relative tolerance
};

struct AdjArgs {
  const DevModel* mdl;
  int64_t P;
  double dtau;
  const double *rho11, *chi0, *theta;
  const double *D, *ye, *e;
  const int32_t *status, *n_outer;
  const double* gbar;
  double* grad_pp;     // (P, nq + 2) per-point terms or nullptr
  double* partial;       // (work-groups of the iteration, nq + 2) partial sums
  double* partial_left;  // (work-groups of the elimination, nq + 2) likewise, written where `had` is set
  uint8_t* had;          // per work-group of the elimination: whether it had a point (kAdjPartials bytes)
  uint8_t* left;       // per pair of points: bit h set where half h is left to the elimination
};

// Work-groups of the adjoint's two kernels.  Two per SIMD stay resident; the
// elimination's unevenly loaded ones are twice as many in long batches (65536
// points, all eliminated, 2086 against 2151 us; 4096 points, none, 39.6 against
// 37.4 us).
struct AdjGrid {
  int64_t iterate, eliminate;
};
inline AdjGrid adj_grid(int64_t P, int num_cu) {
  const int64_t pairs = (P + 1) / 2, resident = (int64_t)num_cu * 8;
  AdjGrid g = {resident, P > 4 * resident ? 2 * resident : resident};
  if (g.iterate > kAdjPartials) g.iterate = kAdjPartials;
  if (g.eliminate > kAdjPartials) g.eliminate = kAdjPartials;
  if (g.iterate > pairs) g.iterate = pairs;
  if (g.eliminate > P) g.eliminate = P;
  return g;
}

// How a solve over `units` (points, or pairs of points) is launched.
struct LaunchPlan {
  int64_t grid;
  int chunk;   // units per work-group or queue grab
  bool queue;  // persistent grid with the work queue
};

// Plan of a solve kernel that keeps `per_cu` work-groups resident per compute
// unit.  A persistent launch takes its units from the work queue once the
// batch is longer than `rounds` rounds of the resident work-groups.
// Below that every unit gets a work-group of its own and the hardware
// dispatcher is the queue: it starts the next unit wherever one ends, with no
// counters to reset and no ticket to wait for (a caller that limits
// blocks_per_cu keeps the queue).  Measured, one unit per grab, direct
// against queue: static solve of 4095 points (1 round) 74 against 80 us, 16384
// points (4 rounds) 115 against 141 us, 65536 points (16 rounds) 398 against
// 409 us; 64 nodes, 8192 points (4 rounds) 125 against 150 us, 32768 points (16
// rounds) 434 against 450 us, 131072 points (64 rounds) 1726 against 1728 us.
// The coupled O(v) kernel, alone on its SIMD, has no other wave to cover the
// start of a work-group (model tables, inputs), and a queue's waves load the
// tables once: 4096 points (2 rounds) 241 against 247 us, 8192 points (4
// rounds) 415 against 414, 16384 points 774 against 775, 32768 points 1500
// against 1488; with linear-order kernels 4096 points 401 against 406, 8192
// points 683 against 677, 16384 points 1277 against 1266, 32768 points 2476
// against 2441.
// A grab takes at most 1/64 of a work-group's even share of the batch (among
// the caller's work-groups where blocks_per_cu sets them), whatever chunk
// allows, so that no work-group is left with several units
// when the others are done (4 pairs per grab: 4095 points 320 us, one: 95 us).
constexpr int64_t kDirectRounds = 16, kDirectRoundsV = 4;
inline LaunchPlan plan_launch(const nmc_launch& L, int64_t units, int per_cu, int num_cu,
                              int64_t rounds = kDirectRounds) {
  LaunchPlan p = {0, L.chunk, false};
  if (L.persistent) {
    const int64_t slots = (int64_t)per_cu * num_cu;
    p.queue = L.blocks_per_cu > 0 || units > rounds * slots;
    const int64_t groups = L.blocks_per_cu > 0 ? (int64_t)L.blocks_per_cu * num_cu : slots;
    const int64_t share = p.queue ? units / (64 * groups) : 1;
    if (p.chunk > share) p.chunk = share > 1 ? (int)share : 1;
  }
  p.grid = (units + p.chunk - 1) / p.chunk;
  if (p.queue) {
    // a surplus of work-groups over the resident ones is harmless: late ones
    // find the queue drained and exit
    const int64_t most = (int64_t)(L.blocks_per_cu > 0 ? L.blocks_per_cu : 2 * per_cu) * num_cu;
    if (p.grid > most) p.grid = most;
  }
  if (p.grid < 1) p.grid = 1;
  return p;
}

// Whether a batch is small enough for one wavefront per species of a pair of
// points instead of one per pair: up to `waves` such wavefronts per compute
// unit (eight are resident).  There the slowest points set the time and their
// share of work per wavefront is what counts; beyond, the species' common work
// (equation of state, rows) done once per wavefront costs more.  Each number of
// species has a line of its own: with two, a pair's wave has less to share out.
// Mean us over six draws, split against pairs, at the line and beyond it:
// static solve of three species, 3413 points (20 waves) 75 against 77, 4096
// points 87 against 81; projected equilibrium 111 against 122 and 130 against
// 122; two species 4096 points (16 waves) 54 against 54 and projected 79 against
// 82, 4352 points 58 against 55 and 86 against 83.  O(v) solve of three species,
// 2389 points (14 waves) 215 against 230, 2730 points 238 against 220; two
// species 2560 points (10 waves) 129 against 132, 2816 points 135 against 133.
// With linear-order kernels three species 2730 points (16 waves) 348 against
// 374, 3072 points 386 against 376; two species 2816 points (11 waves) 200
// against 208, 3072 points 217 against 213.  Small batches: static solve of 8
// points 44 against 61, O(v) 119 against 173, with linear-order kernels 168
// against 289.  The two kernels give the same bits, so results do not depend on
// the batch; kernel_store = PAIRED keeps the two-point kernel.
constexpr int split_waves(int ns) { return ns == 2 ? 16 : 20; }
constexpr int split_waves_v(int ns, bool phi1) { return phi1 ? (ns == 2 ? 11 : 16) : (ns == 2 ? 10 : 14); }
inline bool split_by_species(const nmc_launch& L, int64_t P, int ns, int num_cu, int waves) {
  return L.kernel_store == NMC_KERNELS_ON_CHIP && ns > 1 && (P + 1) / 2 * ns <= (int64_t)waves * num_cu;
}

// its grid: one work-group per pair, or as many as the caller wants resident
// or per chunk, each taking every gridDim.x-th pair
inline int64_t split_grid(const nmc_launch& L, int64_t P, int num_cu) {
  const int64_t pairs = (P + 1) / 2;
  int64_t grid = pairs;
  if (L.persistent && L.blocks_per_cu > 0) grid = (int64_t)L.blocks_per_cu * num_cu;
  if (!L.persistent) grid = (pairs + L.chunk - 1) / L.chunk;
  return grid < pairs ? grid : pairs;
}

// launchers (defined in the kernel translation units)
hipError_t launch_forward(const FwdArgs& a, int nq, int ns, bool coupled, bool proj, const nmc_launch& L,
                          int num_cu, hipStream_t s);
hipError_t launch_forward64(const FwdArgs& a, int ns, bool coupled, const nmc_launch& L, int num_cu,
                            hipStream_t s);
hipError_t launch_forward_pair(const FwdArgs& a, int ns, bool coupled, bool proj, const nmc_launch& L,
                               int num_cu, hipStream_t s);
hipError_t launch_forward_split(const FwdArgs& a, int ns, bool proj, const nmc_launch& L, int num_cu, hipStream_t s);
hipError_t launch_forward_vsplit(const FwdVArgs& a, int ns, bool phi1, const nmc_launch& L, int num_cu, hipStream_t s);
hipError_t launch_forward_v(const FwdVArgs& a, int ns, bool coupled, bool phi1, const nmc_launch& L, int num_cu,
                            hipStream_t s);
hipError_t launch_forward_vpair(const FwdVArgs& a, int ns, bool coupled, bool phi1, const nmc_launch& L, int num_cu,
                                hipStream_t s);
hipError_t launch_reset_counter(int* counter, hipStream_t s);
hipError_t launch_c2p(int64_t P, int ns, int nq, const double* N, const double* G, const double* v, int mem,
                      double tol, int max_it, double* D, double* I, int32_t* iters, int num_cu, hipStream_t s);
hipError_t launch_pdars_stage3(const PdarsArgs& a, int num_cu, hipStream_t s);
hipError_t launch_pdars_merge(int64_t P, int nn, const int32_t* no2, const int32_t* ni2, const int32_t* st2,
                              const int32_t* iters, int32_t* n_outer, int32_t* n_inner, int32_t* status, int num_cu,
                              hipStream_t s);
// near-equilibrium initial state from raw draws
hipError_t launch_init_state(const DevModel* mdl, int ns, int nq, int64_t P, const double* T, const double* mu,
                             const double* rho11, const double* ye, const double* uD, const double* uI, double a,
                             double b, double c, double* D0, double* I0, double* e0, hipStream_t s);
// adds the sum over points to grad_theta (nq + 2)
hipError_t launch_adjoint(const AdjArgs& a, int nq, int ns, int num_cu, double* grad_theta, hipStream_t s);

}  // namespace nmc
