"""A point's result does not depend on the size of its batch: the small-batch
kernels (one wavefront per species of a pair of points) give the same bits as
the two-points-per-wavefront kernels of larger batches, every output and every
count, for every option of the solve, at single points, odd batches, the last
batch that is split and the first that is not (for each number of species and
kernel its own), and at points that are cold, skipped, capped or fail, in every
pairing with warm ones.  The larger batch holds the same points repeated, so
that its pairs are the small batch's."""
import numpy as np
import pytest

from paper_2601_00976_amd import native as N
from paper_2601_00976_amd import solver as S
from paper_2601_00976_amd import workloads as W

pytestmark = pytest.mark.gpu

SP3 = (N.NU_E, N.NU_E_BAR, N.NU_X)
SP2 = (N.NU_E, N.NU_E_BAR)


def _line(ns, waves):
    """Points of the largest batch that is split: `waves` wavefronts per compute unit, one per species and pair."""
    import torch
    return 2 * (waves * torch.cuda.get_device_properties(0).multi_processor_count // ns)


def _same_bits(run, t, P):
    import torch
    a = run(t)
    b = run({k: v.repeat((-(-8194 // P),) + (1,) * (v.dim() - 1)) for k, v in t.items()})
    torch.cuda.synchronize()
    for k in a:
        x, y = a[k], b[k][:P]
        assert bool(((x == y) | ((x != x) & (y != y))).all()), (k, int((x != y).sum()))
    return a


def _static(m, d, chi0=None):
    import torch
    t = S.to_device(d)
    D0, I0, e0 = S.init_state(m, t["T"], t["rho11"], t["ye"], t["uD"], t["uI"])
    return dict(D0=D0, I0=I0, rho=t["rho11"], ye=t["ye"], e0=e0, T=t["T"], mu=5.0 * torch.ones_like(t["rho11"]),
                chi0=(chi0 or 1.0) * t["rho11"])


def _solve(m, prm, chi0=False):
    def run(t):
        fixed = dict(T_fixed=t["T"], mu_fixed=t["mu"]) if prm.fixed_matter else {}
        return S.solve(m, prm, W.DTAU_KM, t["D0"], t["I0"], t["rho"], t["ye"], t["e0"], m.default_theta(),
                       chi0=t["chi0"] if chi0 else None, **fixed)
    return run


OPTIONS = [(SP3, {}), (SP2, {}), (SP3, {"fd_projection": 1}), (SP2, {"fd_projection": 1}),
           (SP3, {"flags": N.EMAB | N.NES}), ((N.NU_X, N.NU_E_BAR, N.NU_E), {})]


@pytest.mark.parametrize("P", [1, 2, 77, "line", "line + 1"])
@pytest.mark.parametrize("sp,options", OPTIONS)
def test_static(P, sp, options):
    P = P if isinstance(P, int) else _line(len(sp), {2: 16, 3: 20}[len(sp)]) + (P != "line")
    print(f"[case] static solve by batch size, P={P} species {sp} {options}", flush=True)
    m = S.Model(S.Grid(16), species=sp, **options)
    d = W.radial_profile(P=1 << 16, ns=len(sp), seed=11).take(np.linspace(3000, 60000, P).astype(np.int64))
    t = _static(m, d)
    for prm in (S.Params(), S.Params(m_inner=1, m_outer=2), S.Params(m_inner=2, max_inner=3), S.Params(max_outer=2)):
        _same_bits(_solve(m, prm), t, P)


@pytest.mark.parametrize("options", [{}, {"fd_projection": 1}])
def test_static_cold_failing_and_fixed(options):
    """T 0.05-2 MeV in one batch, on both sides of every line at which the pair factors change their form."""
    import torch
    print(f"[case] static solve by batch size, cold and failing points, {options}", flush=True)
    m = S.Model(S.Grid(16), **options)
    P = 96
    d = W.radial_profile(P=1 << 16, seed=3).take(np.linspace(20000, 44000, P).astype(np.int64))
    T = np.random.default_rng(5).permutation(np.concatenate([np.geomspace(0.05, 0.3, P // 2), np.geomspace(0.3, 2.0, P // 2)]))
    t = _static(m, W.Draws(**{**d.__dict__, "T": T}), chi0=8.0)
    fixed = _same_bits(_solve(m, S.Params(fixed_matter=True), chi0=True), t, P)
    assert bool((fixed["status"] == 0).any())
    _same_bits(_solve(m, S.Params(max_outer=5), chi0=True), t, P)
    t["e0"][3] = t["e0"][40] = -1.0  # no temperature
    t["D0"][7, 0, 5] = t["I0"][20, 2, 31] = float("nan")
    t["rho"][11] = 1e-6  # uncoupled
    out = _same_bits(_solve(m, S.Params(max_outer=5)), t, P)
    assert out["status"][[3, 40]].tolist() == [N.STATUS_EOS_DOMAIN] * 2
    assert out["status"][[7, 20]].tolist() == [N.STATUS_NONFINITE] * 2
    assert int(out["n_outer"][11]) == 0 and int(out["status"][11]) == 0


PRM = dict(tol_inner=1e-12, tol_outer=1e-10)
PHI1 = dict(phi1_nes=0.3, phi1_pair=-0.25)


def _moving(m, d):
    t = S.to_device(d)
    D0, I0, ef0 = S.init_state_v(m, t)
    return dict(D0=D0, I0=I0, rho=t["rho11"], ye=t["ye"], ef=ef0, v=t["v"])


def _solve_v(m, prm):
    return lambda t: S.solve_v(m, prm, W.DTAU_KM, t["D0"], t["I0"], t["rho"], t["ye"], t["ef"], t["v"],
                               m.default_theta())


@pytest.mark.parametrize("P", [1, 2, 77, "line", "line + 1"])
@pytest.mark.parametrize("sp,options", [(SP3, {}), (SP2, {}), (SP3, PHI1), (SP2, PHI1),
                                        (SP3, {"flags": N.EMAB | N.NES}), ((N.NU_X, N.NU_E_BAR, N.NU_E), {})])
def test_moving(P, sp, options):
    P = P if isinstance(P, int) else _line(len(sp), ({2: 11, 3: 16} if options == PHI1 else {2: 10, 3: 14})[len(sp)]) + (P != "line")
    print(f"[case] O(v) solve by batch size, P={P} species {sp} {options}", flush=True)
    m = S.Model(S.Grid(16), species=sp, **options)
    t = _moving(m, W.radial_profile_v(P=1 << 16, ns=len(sp)).take(np.linspace(4000, 55000, P).astype(np.int64)))
    for prm in (S.Params(**PRM), S.Params(m_inner=1, m_outer=2, max_outer=4, **PRM), S.Params(m_inner=2, max_inner=3, **PRM),
                S.Params(fixed_matter=True, **PRM)):
        _same_bits(_solve_v(m, prm), t, P)


@pytest.mark.parametrize("options", [{}, PHI1])
def test_moving_cold_and_failing(options):
    import torch
    print(f"[case] O(v) solve by batch size, cold and failing points, {options}", flush=True)
    m = S.Model(S.Grid(16), **options)
    P = 96
    d = W.radial_profile_v(P=1 << 16).take(np.linspace(20000, 44000, P).astype(np.int64))
    T = np.random.default_rng(5).permutation(np.concatenate([np.geomspace(0.05, 0.3, P // 2), np.geomspace(0.3, 2.0, P // 2)]))
    t = _moving(m, W.Draws(**{**d.__dict__, "T": T}))
    fixed = _same_bits(_solve_v(m, S.Params(fixed_matter=True, **PRM)), t, P)
    assert bool((fixed["status"] == 0).any())
    _same_bits(_solve_v(m, S.Params(max_outer=5, **PRM)), t, P)
    t["ef"][3] = t["ef"][40] = -1.0  # no temperature
    t["D0"][7, 0, 5] = t["I0"][20, 2, 1, 31] = float("nan")
    t["rho"][11] = 1e-6  # uncoupled
    t["I0"][12] = 0.0
    t["v"][13] = 0.0
    out = _same_bits(_solve_v(m, S.Params(max_outer=5, **PRM)), t, P)
    assert out["status"][[3, 40]].tolist() == [N.STATUS_EOS_DOMAIN] * 2
    assert out["status"][[7, 20]].tolist() == [N.STATUS_NONFINITE] * 2
    assert int(out["n_outer"][11]) == 0 and int(out["status"][11]) == 0
