"""The 64-node solve's row of the symmetric core in registers and the columns
regenerated at colder points: temperatures on both sides of the line between
them (~0.22 MeV on the 1-300 MeV grid) in one batch, every number of species.
The stored core gives the same bits, and the warm points agree with the oracle
to the parity tests' bar."""
import numpy as np
import pytest

import oracle as O
from paper_2601_00976_amd import native as N
from paper_2601_00976_amd import solver as S
from paper_2601_00976_amd import workloads as W
from tests import parity as PT
from tests.test_gpu_parity import _compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sp", [(O.NU_E, O.NU_E_BAR, O.NU_X), (O.NU_E, O.NU_E_BAR), (O.NU_X,)])
def test_rows_and_regenerated_columns(sp):
    import torch
    print(f"[case] 64 nodes, T 0.1-3 MeV in one batch, species {sp}", flush=True)
    ns, P = len(sp), 61
    d = W.radial_profile(P=1 << 16, ns=ns, nq=64, seed=7).take(np.linspace(20000, 40000, P).astype(np.int64))
    T = np.where(np.arange(P) % 3 == 0, np.linspace(0.1, 0.4, P), np.linspace(0.5, 3.0, P))
    d = W.Draws(**{**d.__dict__, "T": T})
    theta = np.concatenate([np.ones(64), [PT.A_NES, PT.A_PAIR]])
    m, ref = PT.run_oracle(d, sp, O.ALL_PHYSICS, W.DTAU_KM, O.Params(), theta, n_elem=32)
    _, got = PT.run_gpu(d, sp, O.ALL_PHYSICS, W.DTAU_KM, S.Params(), theta, n_elem=32)
    warm = np.flatnonzero(T >= 0.5)
    pick = lambda r: {k: v[warm] for k, v in r.items()}
    _compare(pick(ref), pick(got), m.w2, model=m, rho11=d.rho11[warm], species=sp)
    mg = S.Model(S.Grid(32), species=sp)
    t = S.to_device(d)
    D0, I0, e0 = S.init_state(mg, t["T"], t["rho11"], t["ye"], t["uD"], t["uI"])
    ws = S.Workspace(mg, P, kernel_store=True)
    b = S.solve(mg, S.Params(), W.DTAU_KM, D0, I0, t["rho11"], t["ye"], e0, torch.as_tensor(theta, device="cuda"),
                workspace=ws, launch=S.LaunchConfig(kernel_store=N.KERNELS_HBM))
    torch.cuda.synchronize()
    for k in b:
        assert np.array_equal(got[k], b[k].cpu().numpy()), k
