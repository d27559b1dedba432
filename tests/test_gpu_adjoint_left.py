"""Points that the adjoint's iteration leaves to the elimination: they fall
behind early instead of using up the iterations, two of a pair are eliminated
side by side, and the sums over the work-groups that had any are right and the
same in every call.  The per-point terms themselves are pinned by the route
tests against the dense-LU oracle; here the batch is large enough for every
work-group to take several points."""
import numpy as np
import pytest

from paper_2601_00976_amd import solver as S
from paper_2601_00976_amd import workloads as W

pytestmark = pytest.mark.gpu


def _case(d, dtau):
    """Forward solve of the draws and the adjoint of it as a call."""
    import torch
    m = S.Model(S.Grid(16))
    t = S.to_device(d)
    D0, I0, e0 = S.init_state(m, t["T"], t["rho11"], t["ye"], t["uD"], t["uI"])
    theta = m.default_theta()
    out = S.solve(m, S.Params(max_inner=1000, max_outer=200), dtau, D0, I0, t["rho11"], t["ye"], e0, theta)
    gbar = torch.as_tensor(np.random.default_rng(1).uniform(-1, 1, (d.P, 2)), device="cuda")
    ws, g = S.Workspace(m, d.P), torch.zeros(34, dtype=torch.float64, device="cuda")

    def call(**kw):
        return S.adjoint(m, dtau, t["rho11"], theta, out, gbar, workspace=ws, **kw)
    return call, lambda: call(grad_theta=g), out


def _us(call):
    """Shortest of many mean times over ten calls."""
    import torch
    a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    best = float("inf")
    for _ in range(30):
        a.record()
        for _ in range(10):
            call()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 100)
    return best


def _stiff(P):
    return W.radial_profile(P=1 << 16).take(np.linspace(0, 800, P).astype(np.int64))


def test_left_points_side_by_side():
    print("[case] adjoint: two stiff points take no longer than one", flush=True)
    one, two = (_us(_case(_stiff(P), 0.5)[1]) for P in (1, 2))
    print(f"one {one:.1f} us, two {two:.1f} us", flush=True)
    assert two <= 1.2 * one


def test_left_points_do_not_use_up_the_iterations():
    """Against a point too cold for the iteration, which goes to the elimination at once."""
    print("[case] adjoint: a stiff point falls behind early", flush=True)
    d = _stiff(1)
    cold = W.Draws(**{**d.__dict__, "T": np.full(1, 0.15), "rho11": np.full(1, 1.0)})
    stiff, at_once = _us(_case(d, 0.5)[1]), _us(_case(cold, 1e-3)[1])
    print(f"stiff {stiff:.1f} us, cold {at_once:.1f} us", flush=True)
    assert stiff <= 1.4 * at_once


@pytest.mark.parametrize("P", [1, 3, 4095, 4097, 9001])
def test_sums_over_both_kernels(P):
    import torch
    print(f"[case] adjoint: sums over the work-groups of both kernels, P={P}", flush=True)
    idx = np.random.default_rng(P).permutation(np.linspace(0, 60000, P).astype(np.int64))  # stiff, settled, skipped
    call, _, out = _case(W.radial_profile(P=1 << 16).take(idx), 0.5)
    g, gpp = call(per_point=True)
    again = [call() for _ in range(3)]
    torch.cuda.synchronize()
    for x in again:
        assert torch.equal(x, g)
    dead = (out["status"] != 0) | (out["n_outer"] == 0)
    assert bool((gpp[dead] == 0.0).all())
    scale = gpp.abs().sum(0)
    # two orders of adding P terms: each rounds at most P times by 2^-53 of the sum of magnitudes
    assert bool(((gpp.sum(0) - g).abs() <= 2 * P * 2.0 ** -53 * scale).all())
