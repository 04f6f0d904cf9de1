"""Forward sweeps whose windows are whole lines of padded rows (large batches at
the default tile depth): every source comes out as from slabs of any depth, bit
for bit, at rows one node either side of a line, ragged tile columns, and
without the workspace for them."""
import numpy as np
import pytest

from paper_2412_00031_amd import api
from paper_2412_00031_amd import workloads as W

pytestmark = pytest.mark.gpu

COLUMNS = 3072  # tile columns of a batch from which on the fields are padded


# n2 = 16 q - 1 .. 16 q + 2 (the last line full, its k face alone on a line, one and two
# nodes over), a row within one line, several lines; one tile column, ragged ones, several
@pytest.mark.parametrize("n", [(10, 10, 4), (9, 10, 15), (10, 7, 16), (5, 9, 17), (10, 10, 18), (11, 19, 31),
                               (18, 10, 33), (4, 4, 47), (20, 27, 50)])
def test_lines_equal_slabs(torch_cuda, n):
    torch = torch_cuda
    cols = ((n[0] + 5) // 8) * ((n[1] + 5) // 8)
    nsrc = -(-COLUMNS // cols)
    wl = W.small_spherical(n=n, nsrc=4, nrec=2, seed=sum(n))
    g, kap = wl["grid"], wl["kappa"]
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    s, xi, eta, src = (t(wl[k]) for k in ("s", "xi", "eta", "src"))
    src = src.repeat(-(-nsrc // 4), 1)[:nsrc].contiguous()
    par = api.source_params(g, s, xi, eta, src)
    tau, st = api.forward(g, s, xi, eta, src, par, 1e-8, 400, kap, poll=True)
    one = slice(0, 4)
    ref, sr = api.forward(g, s, xi, eta, src[one].contiguous(), par[one].contiguous(), 1e-8, 400, kap, poll=True, tile_k=5)
    assert (sr > 0).all()
    for q in (*range(4), nsrc - 4, nsrc - 1):
        assert int(st[q]) == int(sr[q % 4]) and torch.equal(tau[q], ref[q % 4]), q
    # warm start in place, and a workspace without the padded fields
    ws = api.workspace(g, nsrc, 0, device="cuda")
    small = ws[: ws.numel() - 8 * nsrc * n[0] * n[1] * n[2]].contiguous()
    tau2, st2 = api.forward(g, s, xi, eta, src, par, 1e-8, 400, kap, poll=True, tau_init=tau)
    tau3, st3 = api.forward(g, s, xi, eta, src, par, 1e-8, 400, kap, poll=True, ws=small)
    ref2, _ = api.forward(g, s, xi, eta, src[one].contiguous(), par[one].contiguous(), 1e-8, 400, kap, poll=True, tile_k=5,
                          tau_init=tau[one].contiguous())
    assert torch.equal(tau2[one], ref2) and torch.equal(tau3, tau) and torch.equal(st3, st)


def test_fewer_groups_where_the_workspace_holds_fewer(torch_cuda):
    """The default number of groups needs a workspace per group; one that was
    sized for a single group serves the call all the same."""
    torch = torch_cuda
    n, nsrc = (20, 27, 12), 128  # 1536 tile columns: two groups forward, four adjoint
    wl = W.small_spherical(n=n, nsrc=nsrc, nrec=3, seed=5)
    g, kap = wl["grid"], wl["kappa"]
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    s, xi, eta, src, rec, R = (t(wl[k]) for k in ("s", "xi", "eta", "src", "rec", "R"))
    par = api.source_params(g, s, xi, eta, src)
    tau, st = api.forward(g, s, xi, eta, src, par, 1e-8, 400, kap, poll=True)
    lam, sa = api.adjoint(g, s, xi, eta, src, par, tau, rec, R, 1e-8, 400, kap, poll=True)
    w0, w1 = (api.workspace(g, nsrc, q, device="cuda", groups=1) for q in (0, 1))
    tau1, st1 = api.forward(g, s, xi, eta, src, par, 1e-8, 400, kap, poll=True, ws=w0)
    lam1, sa1 = api.adjoint(g, s, xi, eta, src, par, tau, rec, R, 1e-8, 400, kap, poll=True, ws=w1)
    assert torch.equal(tau1, tau) and torch.equal(st1, st) and torch.equal(lam1, lam) and torch.equal(sa1, sa)
