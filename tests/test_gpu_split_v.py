"""The O(v) small-batch kernels (one wavefront per species of a pair of
points) against the two-points-per-wavefront kernels, which the oracle tests
pin, with the measures, the bound (1e-9) and the status rule of those tests (a
point whose outer iteration stalls at its noise floor may end with MAX_OUTER
on one side only).  Odd batches, single points, cold and skipped points next
to warm ones, every option of the solve, the last batch that is split and the
first that is not; and bitwise the same answer for a point whatever its
neighbour, its half and the launch.  The two-points-per-wavefront answer is
that of the same points in a batch large enough for it."""
import numpy as np
import pytest

import oracle as O
from paper_2601_00976_amd import native as N
from paper_2601_00976_amd import solver as S
from paper_2601_00976_amd import workloads as W
from tests import parity as PT

pytestmark = pytest.mark.gpu

SP3 = (N.NU_E, N.NU_E_BAR, N.NU_X)
SP2 = (N.NU_E, N.NU_E_BAR)
PRM = dict(tol_inner=1e-12, tol_outer=1e-10)
PHI1 = dict(phi1_nes=0.3, phi1_pair=-0.25)

TOL = 1e-9


def _same(a, b, m, sp, rho11):
    a, b = ({k: v.cpu().numpy() for k, v in x.items()} for x in (a, b))
    either = (a["status"] == N.STATUS_MAX_OUTER) | (b["status"] == N.STATUS_MAX_OUTER)
    assert np.array_equal(a["status"][~either], b["status"][~either])
    ok = (a["status"] == 0) & (b["status"] == 0)
    assert ok.mean() > 0.9
    errs = PT.parity_errors_v({k: v[ok] for k, v in b.items()}, {k: v[ok] for k, v in a.items()}, m.grid.w2, m.grid.w3,
                              O.Model().c.kcoup, rho11[ok], species=sp)
    assert max(e.max() for e in errs) <= TOL


def _draws(idx, ns):
    return W.radial_profile_v(P=1 << 16, ns=ns).take(idx)


def _state(m, d):
    t = S.to_device(d)
    D0, I0, ef0 = S.init_state_v(m, t)
    return dict(D0=D0, I0=I0, rho=t["rho11"], ye=t["ye"], ef=ef0, v=t["v"])


def _in_a_large_batch(run, t, P):
    """run(t) of the points of t repeated to at least 8192 points, the first P of the results"""
    big = {k: v.repeat((-(-8192 // P),) + (1,) * (v.dim() - 1)) for k, v in t.items()}
    return {k: v[:P] for k, v in run(big).items()}


@pytest.mark.parametrize("P", [1, 2, 3, 77, 2047, 2049])
@pytest.mark.parametrize("sp,options", [(SP3, {}), (SP3, PHI1), (SP2, PHI1), (SP3, {"flags": N.EMAB | N.NES}),
                                        ((N.NU_X, N.NU_E_BAR, N.NU_E), {})])
def test_split_moving(P, sp, options):
    import torch
    print(f"[case] split O(v) P={P} species {sp} {options}", flush=True)
    m = S.Model(S.Grid(16), species=sp, **options)
    lo, hi = (4000, 35000) if P <= 3 else (4000, 55000)  # the larger batches end in skipped points
    d = _draws(np.linspace(lo, hi, P).astype(np.int64), len(sp))
    t = _state(m, d)
    run = lambda t, prm, **kw: S.solve_v(m, prm, W.DTAU_KM, t["D0"], t["I0"], t["rho"], t["ye"], t["ef"], t["v"],
                                         m.default_theta(), **kw)
    prms = [S.Params(**PRM), S.Params(fixed_matter=True, **PRM)]
    if P <= 77:
        prms += [S.Params(m_inner=1, m_outer=2, max_inner=300, **PRM)]
    for prm in prms:
        a, b = run(t, prm), _in_a_large_batch(lambda x: run(x, prm), t, P)
        torch.cuda.synchronize()
        _same(a, b, m, sp, d.rho11)
    if P > 3:  # on other launches, and shifted by one point (every point in its other half, with another neighbour)
        a, c = run(t, prms[0]), run(t, prms[0], launch=S.LaunchConfig(blocks_per_cu=1))
        b = run({k: v[1:].contiguous() for k, v in t.items()}, prms[0])
        torch.cuda.synchronize()
        for k in a:
            assert torch.equal(a[k], c[k]), k
            assert P > 2048 or torch.equal(a[k][1:], b[k]), k


@pytest.mark.parametrize("options", [{}, PHI1])
def test_split_moving_cold(options):
    """Some points colder than the rows in registers allow (0.2 MeV), alone in
    a pair, together, and next to a warm one, at fixed matter (the coupled
    problem has no stable solution that cold)."""
    import torch
    print(f"[case] split O(v), T from 0.08 MeV, {options}", flush=True)
    m = S.Model(S.Grid(16), **options)
    P = 41
    d = _draws(np.linspace(8000, 40000, P).astype(np.int64), 3)
    k = np.arange(P)
    d.T = np.where((k % 3 == 0) | (k > 34), np.linspace(0.08, 0.2, P), d.T)
    t = _state(m, d)
    run = lambda t: S.solve_v(m, S.Params(fixed_matter=True, **PRM), W.DTAU_KM, t["D0"], t["I0"], t["rho"], t["ye"],
                              t["ef"], t["v"], m.default_theta())
    a, b = run(t), _in_a_large_batch(run, t, P)
    torch.cuda.synchronize()
    _same(a, b, m, SP3, d.rho11)
