"""The launch plan's two routes (one work-group per unit, work queue) give the
same bits at every size where the plan can go wrong: single points, odd
batches, the last direct size and the first queued one."""
import pytest

from paper_2601_00976_amd import native as N
from paper_2601_00976_amd import solver as S
from paper_2601_00976_amd import workloads as W

pytestmark = pytest.mark.gpu

LINE = 16 * 8 * 256  # units (points, or pairs of points) of the last direct launch on 256 compute units


def _solve(m, t, state, theta, launch):
    D0, I0, e0 = state
    return S.solve(m, S.Params(), W.DTAU_KM, D0, I0, t["rho11"], t["ye"], e0, theta, launch=launch)


@pytest.mark.parametrize("n_elem,P", [(16, 1), (16, 3), (16, 2 * LINE - 1), (16, 2 * LINE + 1), (32, 1), (32, LINE),
                                      (32, LINE + 1)])
def test_direct_and_queued_launches_bitwise(n_elem, P):
    import torch
    print(f"[case] launch plan, {2 * n_elem} nodes, P={P}", flush=True)
    m = S.Model(S.Grid(n_elem))
    t = S.to_device(W.radial_profile(P=P, nq=2 * n_elem, seed=5))
    state = S.init_state(m, t["T"], t["rho11"], t["ye"], t["uD"], t["uI"])
    theta = m.default_theta()
    ref = _solve(m, t, state, theta, None)
    for launch in (S.LaunchConfig(blocks_per_cu=8, chunk=4), S.LaunchConfig(chunk=3, persistent=False)):
        got = _solve(m, t, state, theta, launch)
        torch.cuda.synchronize()
        for k in ref:
            assert torch.equal(ref[k], got[k]), (launch, k)


@pytest.mark.parametrize("P", [1, 2 * 4 * 4 * 256 - 1, 2 * 4 * 4 * 256 + 1])
def test_direct_and_queued_launches_bitwise_v(P):
    import torch
    print(f"[case] launch plan, O(v), P={P}", flush=True)
    m = S.Model(S.Grid(16))
    t = S.to_device(W.radial_profile_v(P=P, seed=5))
    D0, I0, ef0 = S.init_state_v(m, t)
    prm = S.Params(tol_inner=1e-12, tol_outer=1e-10)
    args = (m, prm, W.DTAU_KM, D0, I0, t["rho11"], t["ye"], ef0, t["v"], m.default_theta())
    ref = S.solve_v(*args)
    got = S.solve_v(*args, launch=S.LaunchConfig(blocks_per_cu=4, chunk=2))
    torch.cuda.synchronize()
    for k in ref:
        assert torch.equal(ref[k], got[k]), k


def test_kernels_in_hbm_direct_and_queued():
    import torch
    print("[case] launch plan, kernels in HBM, P=77", flush=True)
    P, m = 77, S.Model(S.Grid(32))
    t = S.to_device(W.radial_profile(P=P, nq=64, seed=6))
    D0, I0, e0 = S.init_state(m, t["T"], t["rho11"], t["ye"], t["uD"], t["uI"])
    ws = S.Workspace(m, P, kernel_store=True)
    res = [S.solve(m, S.Params(), W.DTAU_KM, D0, I0, t["rho11"], t["ye"], e0, m.default_theta(), workspace=ws,
                   launch=S.LaunchConfig(blocks_per_cu=b, kernel_store=N.KERNELS_HBM)) for b in (0, 2)]
    torch.cuda.synchronize()
    for k in res[0]:
        assert torch.equal(res[0][k], res[1][k]), k
