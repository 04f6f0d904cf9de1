"""Kernel accumulation takes one node a thread on small grids, two in a row along axis 0
from 200000 nodes on: against the oracle on both sides of the line, with an even and an
odd number of nodes along axis 0, in both coordinate systems."""
import numpy as np
import pytest

import oracle as O
from conftest import rel_inf
from paper_2412_00031_amd import api
from paper_2412_00031_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("coord", [0, 1])
@pytest.mark.parametrize("n", [(50, 64, 62), (49, 64, 64), (50, 63, 64), (4, 200, 251), (5, 199, 203)])
def test_accum_runs(torch_cuda, coord, n):
    torch = torch_cuda
    nsrc = 2
    wl = W.small_spherical(n=n, nsrc=nsrc, nrec=2, seed=sum(n))
    g, kap, src0 = wl["grid"], wl["kappa"], wl["src"]
    if coord == 0:
        f = (src0 - np.array(g["o"])) / (np.array(g["h"]) * (np.array(n) - 1))
        g, kap = dict(n=n, coord=0, o=(0.0, 0.0, 0.0), h=(1.0, 1.0, 1.0)), 1.0
        src0 = f * (np.array(n) - 1)
    rng = np.random.default_rng(n[2])
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    s, xi, eta, src = (t(v) for v in (wl["s"], wl["xi"], wl["eta"], src0))
    par = api.source_params(g, s, xi, eta, src)
    tau = 1.0 + 0.1 * rng.uniform(-1, 1, (nsrc,) + n)
    lam = rng.normal(size=(nsrc,) + n)
    ref = np.zeros((3,) + n)
    for q in range(nsrc):
        O.kernel(g, wl["s"], wl["xi"], wl["eta"], src0[q], par[q].cpu().numpy(), kap, tau[q], lam[q], ref)
    grad = api.kernel(g, s, xi, eta, src, par, t(tau), t(lam))
    # a few dozen roundings a term, sums of two: the other parity tests' bound is far above
    assert rel_inf(grad.cpu().numpy(), ref) <= 1e-11
