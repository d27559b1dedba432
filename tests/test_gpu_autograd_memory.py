"""A differentiable solve frees its arrays with its outputs: nothing is left to
the cyclic garbage collector, so passes in a loop hold one pass's memory."""
import gc

import pytest

from paper_2601_00976_amd import solver as S
from paper_2601_00976_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("backward", [False, True])
def test_passes_do_not_accumulate(backward):
    import torch
    print(f"[case] memory of repeated passes, backward {backward}", flush=True)
    m = S.Model(S.Grid(16))
    t = S.to_device(W.radial_profile(P=500, seed=2))
    D0, I0, e0 = S.init_state(m, t["T"], t["rho11"], t["ye"], t["uD"], t["uI"])
    theta = m.default_theta().requires_grad_(True)

    def one():
        out = S.NMCSolve.apply(theta, m, S.Params(), W.DTAU_KM, D0, I0, t["rho11"], t["ye"], e0)
        if backward:
            torch.autograd.grad(out[4].sum(), theta)

    gc.collect()
    gc.disable()
    try:
        for _ in range(2):
            one()
        torch.cuda.synchronize()
        held = torch.cuda.memory_allocated()
        for _ in range(5):
            one()
        torch.cuda.synchronize()
        assert torch.cuda.memory_allocated() == held
    finally:
        gc.enable()
