"""Sweep launches hand a batch's tile columns to waves by tickets, in batches of
sources dealt to the XCDs: every source of a batch of any size comes out as it
does alone, bit for bit, forward and adjoint."""
import numpy as np
import pytest

from paper_2412_00031_amd import api
from paper_2412_00031_amd import workloads as W

pytestmark = pytest.mark.gpu


# fewer sources than XCDs, one per XCD, one more, batches past one active mask
# of 64 sources, and past the sources of one launch (512); ragged tile columns
@pytest.mark.parametrize("nsrc,n", [(1, (4, 4, 4)), (3, (11, 10, 9)), (8, (19, 11, 26)), (9, (10, 27, 12)),
                                    (70, (11, 12, 19)), (513, (6, 11, 10)), (1030, (5, 4, 7))])
def test_batch_equals_single_sources(torch_cuda, nsrc, n):
    torch = torch_cuda
    wl = W.small_spherical(n=n, nsrc=nsrc, nrec=6, seed=100 + nsrc)
    g, kap = wl["grid"], wl["kappa"]
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    s, xi, eta, src, rec, R = (t(wl[k]) for k in ("s", "xi", "eta", "src", "rec", "R"))
    par = api.source_params(g, s, xi, eta, src)
    tau, st = api.forward(g, s, xi, eta, src, par, 1e-8, 400, kap, poll=True)
    lam, sa = api.adjoint(g, s, xi, eta, src, par, tau, rec, R, 1e-8, 400, kap, poll=True)
    assert (st > 0).all() and (sa > 0).all()
    picks = sorted({0, nsrc // 2, nsrc - 1, min(7, nsrc - 1), min(64, nsrc - 1), min(511, nsrc - 1), min(512, nsrc - 1)})
    for q in picks:
        one = slice(q, q + 1)
        for tk in (0, 5):
            tau1, st1 = api.forward(g, s, xi, eta, src[one], par[one].contiguous(), 1e-8, 400, kap, poll=True, tile_k=tk)
            lam1, sa1 = api.adjoint(g, s, xi, eta, src[one], par[one].contiguous(), tau1, rec, R[one].contiguous(), 1e-8,
                                    400, kap, poll=True, tile_k=tk)
            assert int(st1[0]) == int(st[q]) and int(sa1[0]) == int(sa[q]), (q, tk)
            assert torch.equal(tau1[0], tau[q]) and torch.equal(lam1[0], lam[q]), (q, tk)
