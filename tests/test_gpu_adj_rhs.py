"""Adjoint right-hand side: receivers are added 64 at a time, nodes shared by
several receivers in receiver order.  The adjoint field of many receivers in few
cells against the oracle."""
import numpy as np
import pytest

import oracle as O
from conftest import rel_inf
from paper_2412_00031_amd import api
from paper_2412_00031_amd import workloads as W

pytestmark = pytest.mark.gpu


# one receiver, a full wave, one more, several waves in a handful of cells; all on the corner node
@pytest.mark.parametrize("nrec,spread", [(1, 1.0), (64, 1.0), (65, 0.3), (200, 0.25), (131, 0.0)])
def test_adjoint_of_crowded_receivers(torch_cuda, nrec, spread):
    torch = torch_cuda
    wl = W.small_spherical(n=(9, 10, 11), nsrc=2, nrec=6, seed=7)
    g, kap = wl["grid"], wl["kappa"]
    rng = np.random.default_rng(nrec)
    far = np.array(g["o"]) + np.array(g["h"]) * (np.array(g["n"]) - 1)
    rec = far - spread * rng.uniform(0, 1, (nrec, 3)) * (far - np.array(g["o"]))
    R = rng.normal(size=(2, nrec))
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    s, xi, eta, src = (t(wl[k]) for k in ("s", "xi", "eta", "src"))
    par = api.source_params(g, s, xi, eta, src)
    tau, st = api.forward(g, s, xi, eta, src, par, 1e-11, 400, kap)
    lam, sa = api.adjoint(g, s, xi, eta, src, par, tau, t(rec), t(R), 1e-11, 400, kap)
    assert (st > 0).all() and (sa > 0).all()
    for q in range(2):
        p = par[q].cpu().numpy()
        rhs = O.adjoint_rhs(g, wl["src"][q], p, rec, R[q])
        ref, it, conv, _ = O.adjoint(g, wl["s"], wl["xi"], wl["eta"], wl["src"][q], p, kap, tau[q].cpu().numpy(), rhs,
                                     1e-11, 400)
        # the same Gauss-Seidel steps: rounding only, the bound of the other parity tests
        assert conv and it == int(sa[q])
        assert rel_inf(lam[q].cpu().numpy(), ref) <= 1e-10
