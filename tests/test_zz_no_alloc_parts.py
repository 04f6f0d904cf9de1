"""tt_forward_noalloc takes every batch whose workspace without the sources' longitude tables
fits its array: one that does not fit with them is solved in parts, bit for bit the
solve in a caller's workspace."""
import numpy as np
import pytest

from paper_2412_00031_amd import api
from paper_2412_00031_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_noalloc_in_parts(torch_cuda):
    torch = torch_cuda
    n, nsrc = (4, 4, 600), 6501
    wl = W.small_spherical(n=n, nsrc=3, nrec=2, seed=9)
    g, kap = wl["grid"], wl["kappa"]
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    s, xi, eta, src = (t(wl[k]) for k in ("s", "xi", "eta", "src"))
    src = src.repeat(nsrc // 3, 1)
    par = api.source_params(g, s, xi, eta, src)
    need = api.workspace(g, nsrc, 0, 28, s.device, groups=1).numel()  # (no padded fields)
    assert need > (64 << 20) + (192 << 10) and need - nsrc * 16 * n[2] < 64 << 20
    ref, ref_st = api.forward(g, s, xi, eta, src, par, 1e-8, 60, kap, groups=1)
    tau, st = torch.full_like(ref, -1.0), torch.full_like(ref_st, 12345)
    api.forward_noalloc(g, s, xi, eta, src, par, 1e-8, 60, kap, tau, st)
    torch.cuda.synchronize()
    assert torch.equal(st, ref_st) and torch.equal(tau, ref)
