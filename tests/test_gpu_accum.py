"""Kernel accumulation takes nodes four at a time along axis 0 and axis 2's
neighbours from the lanes beside: against the oracle at sizes either side of a
thread's run, a wave and a block."""
import numpy as np
import pytest

import oracle as O
from conftest import rel_inf
from paper_2412_00031_amd import api
from paper_2412_00031_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(4, 4, 4), (5, 8, 8), (7, 16, 16), (8, 16, 17), (9, 5, 64), (6, 4, 65)])
def test_accum_sizes(torch_cuda, n):
    torch = torch_cuda
    wl = W.small_spherical(n=n, nsrc=3, nrec=2, seed=sum(n))
    g, kap = wl["grid"], wl["kappa"]
    rng = np.random.default_rng(n[2])
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    s, xi, eta, src = (t(wl[k]) for k in ("s", "xi", "eta", "src"))
    par = api.source_params(g, s, xi, eta, src)
    tau = 1.0 + 0.1 * rng.uniform(-1, 1, (3,) + n)
    lam = rng.normal(size=(3,) + n)
    ref = np.zeros((3,) + n)
    for q in range(3):
        O.kernel(g, wl["s"], wl["xi"], wl["eta"], wl["src"][q], par[q].cpu().numpy(), kap, tau[q], lam[q], ref)
    grad = api.kernel(g, s, xi, eta, src, par, t(tau), t(lam))
    # a few dozen roundings a term, sums of three: the other parity tests' bound is far above
    assert rel_inf(grad.cpu().numpy(), ref) <= 1e-11
    twice = api.kernel(g, s, xi, eta, src, par, t(tau), t(lam), grad=grad.clone())
    assert torch.equal(twice, 2 * grad)
