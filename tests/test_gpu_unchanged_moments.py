"""A point of the O(v) solve that ends before its first inner iteration keeps
its moments, and its matter with them, bit for bit: the old state's Eulerian
integrals and those of the final moments are one function of the same values.
The points fail in the equation of state (an energy below the cold floor) at
densities at the edge of the coupled region, where the matter update multiplies
a difference of the integrals most; every batch size that picks a kernel, alone
in a pair and beside solved points."""
import numpy as np
import pytest

from paper_2601_00976_amd import native as N
from paper_2601_00976_amd import solver as S
from paper_2601_00976_amd import workloads as W

pytestmark = pytest.mark.gpu

SP3 = (N.NU_E, N.NU_E_BAR, N.NU_X)


@pytest.mark.parametrize("P", [1, 64, 8193])
@pytest.mark.parametrize("sp,options", [(SP3, {}), ((N.NU_X,), {}), (SP3, {"flags": N.EMAB | N.ISO}),
                                        (SP3, {"phi1_nes": 0.3, "phi1_pair": -0.25})])
def test_failed_points_keep_their_matter(P, sp, options):
    import torch
    print(f"[case] failed points keep their matter, P={P}, species {sp} {options}", flush=True)
    m = S.Model(S.Grid(16), species=sp, **options)
    d = W.radial_profile_v(P=1 << 16, ns=len(sp)).take(np.linspace(30000, 45000, P).astype(np.int64))
    d = W.Draws(**{**d.__dict__, "rho11": np.geomspace(1.1e-4, 1e-2, P)})
    t = S.to_device(d)
    D0, I0, ef0 = S.init_state_v(m, t)
    bad = torch.arange(P, device="cuda") % 3 != 1
    ef0 = torch.where(bad, torch.full_like(ef0, -1.0), ef0)
    out = S.solve_v(m, S.Params(), W.DTAU_KM, D0, I0, t["rho11"], t["ye"], ef0, t["v"], m.default_theta())
    torch.cuda.synchronize()
    assert bool((out["status"][bad] == N.STATUS_EOS_DOMAIN).all())
    for k, was in (("D", D0), ("I", I0), ("ye", t["ye"]), ("ef", ef0), ("v", t["v"])):
        assert torch.equal(out[k][bad], was[bad]), (k, float((out[k][bad] - was[bad]).abs().max()))
