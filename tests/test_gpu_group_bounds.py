"""Source counts that do not divide by the groups: groups of whole eights, a rest, and
more groups than eights, bit for bit the solve of one group."""
import numpy as np
import pytest

from paper_2412_00031_amd import api
from paper_2412_00031_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nsrc,groups", [(9, 2), (17, 2), (17, 3), (19, 5), (3, 3), (25, 4), (25, 8)])
def test_groups_of_any_split(torch_cuda, nsrc, groups):
    torch = torch_cuda
    wl = W.small_spherical(n=(14, 18, 11), nsrc=nsrc, nrec=3, seed=3)
    g, kap = wl["grid"], wl["kappa"]
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    s, xi, eta, src, rec, R = (t(wl[k]) for k in ("s", "xi", "eta", "src", "rec", "R"))
    par = api.source_params(g, s, xi, eta, src)

    def both(G):
        tau, st = api.forward(g, s, xi, eta, src, par, 1e-8, 400, kap, poll=True, groups=G)
        lam, sa = api.adjoint(g, s, xi, eta, src, par, tau, rec, R, 1e-8, 400, kap, poll=True, groups=G)
        return tau, st, lam, sa

    assert all(torch.equal(a, b) for a, b in zip(both(groups), both(1)))
