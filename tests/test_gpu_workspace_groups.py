"""Workspaces that were sized for fewer source groups than the call asks for: the solve
runs in as many as fit, bit for bit the same; one that holds not even one group's
tables is refused."""
import numpy as np
import pytest

from paper_2412_00031_amd import api
from paper_2412_00031_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sized,asked", [(0, 4), (1, 4), (1, 2), (0, 8)])
def test_workspace_for_fewer_groups(torch_cuda, sized, asked):
    """A workspace sized for fewer groups than the call asks for."""
    torch = torch_cuda
    n = (20, 27, 12)
    for nsrc in (40, 256):  # in place, padded
        wl = W.small_spherical(n=n, nsrc=4, nrec=3, seed=5)
        g, kap = wl["grid"], wl["kappa"]
        t = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
        s, xi, eta, src, rec = (t(wl[k]) for k in ("s", "xi", "eta", "src", "rec"))
        src = src.repeat(nsrc // 4, 1)
        R = t(wl["R"]).repeat(nsrc // 4, 1)
        par = api.source_params(g, s, xi, eta, src)
        tau, st = api.forward(g, s, xi, eta, src, par, 1e-8, 400, kap, poll=True)
        lam, sa = api.adjoint(g, s, xi, eta, src, par, tau, rec, R, 1e-8, 400, kap, poll=True)
        w0, w1 = (api.workspace(g, nsrc, q, device="cuda", groups=sized) for q in (0, 1))
        tau1, st1 = api.forward(g, s, xi, eta, src, par, 1e-8, 400, kap, poll=True, ws=w0, groups=asked)
        lam1, sa1 = api.adjoint(g, s, xi, eta, src, par, tau, rec, R, 1e-8, 400, kap, poll=True, ws=w1, groups=asked)
        assert torch.equal(tau1, tau) and torch.equal(st1, st) and torch.equal(lam1, lam) and torch.equal(sa1, sa)
        with pytest.raises(RuntimeError, match="too small"):
            api.forward(g, s, xi, eta, src, par, 1e-8, 400, kap, poll=True, ws=w0[:1024].contiguous(), groups=asked)
