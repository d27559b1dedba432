"""Queue grabs of several units (the last one ragged, tickets reserved ahead and
taken late) give the bits of one work-group per unit, at every kernel with the
work queue.  One work-group per compute unit, so that 1/64 of its share of the
batch is four units and chunks of 3 and 4 take effect (256 compute units; on
fewer, more)."""
import pytest

from paper_2601_00976_amd import native as N
from paper_2601_00976_amd import solver as S
from paper_2601_00976_amd import workloads as W

pytestmark = pytest.mark.gpu

UNITS = 4 * 64 * 256 + 2


@pytest.mark.parametrize("n_elem,store,per_unit", [(16, N.KERNELS_ON_CHIP, 2), (16, N.KERNELS_WAVE, 1), (32, N.KERNELS_ON_CHIP, 1)])
@pytest.mark.parametrize("chunk", [3, 4])
def test_static(n_elem, store, per_unit, chunk):
    import torch
    P = UNITS * per_unit - (per_unit - 1)
    print(f"[case] queue grabs of {chunk}, {2 * n_elem} nodes, kernel_store {store}, P={P}", flush=True)
    m = S.Model(S.Grid(n_elem))
    t = S.to_device(W.radial_profile(P=P, nq=2 * n_elem, seed=4))
    D0, I0, e0 = S.init_state(m, t["T"], t["rho11"], t["ye"], t["uD"], t["uI"])
    run = lambda L: S.solve(m, S.Params(), W.DTAU_KM, D0, I0, t["rho11"], t["ye"], e0, m.default_theta(), launch=L)
    a = run(S.LaunchConfig(chunk=1, persistent=False, kernel_store=store))
    b = run(S.LaunchConfig(chunk=chunk, blocks_per_cu=1, kernel_store=store))
    torch.cuda.synchronize()
    for k in a:
        assert torch.equal(a[k], b[k]), k


@pytest.mark.parametrize("store,per_unit", [(N.KERNELS_ON_CHIP, 2), (N.KERNELS_WAVE, 1)])
@pytest.mark.parametrize("chunk", [3, 4])
def test_moving(store, per_unit, chunk):
    import torch
    P = UNITS * per_unit - (per_unit - 1)
    print(f"[case] queue grabs of {chunk}, O(v), kernel_store {store}, P={P}", flush=True)
    m = S.Model(S.Grid(16))
    t = S.to_device(W.radial_profile_v(P=P, seed=4))
    D0, I0, ef0 = S.init_state_v(m, t)
    prm = S.Params(tol_inner=1e-12, tol_outer=1e-10, max_outer=8)
    run = lambda L: S.solve_v(m, prm, W.DTAU_KM, D0, I0, t["rho11"], t["ye"], ef0, t["v"], m.default_theta(), launch=L)
    a = run(S.LaunchConfig(chunk=1, persistent=False, kernel_store=store))
    b = run(S.LaunchConfig(chunk=chunk, blocks_per_cu=1, kernel_store=store))
    torch.cuda.synchronize()
    for k in a:
        assert torch.equal(a[k], b[k]), k
