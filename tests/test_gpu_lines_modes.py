"""Padded solves (forward batches whose windows are whole lines) in Cartesian
coordinates, asynchronous, replayed from the library's graphs and from a caller's
graph: bit for bit what slabs give."""
import numpy as np
import pytest

from paper_2412_00031_amd import api
from paper_2412_00031_amd import workloads as W

pytestmark = pytest.mark.gpu

COLUMNS = 3072


def _problem(torch, coord, n, seed, nrec=2):
    wl = W.small_spherical(n=n, nsrc=4, nrec=nrec, seed=seed)
    g = wl["grid"]
    if coord == 0:  # the same model on Cartesian nodes
        pos = wl["src"].copy()
        for a in range(3):
            pos[:, a] = 1.5 * (pos[:, a] - g["o"][a]) / g["h"][a]
        g = dict(n=n, coord=0, o=(0.0, 0.0, 0.0), h=(1.5, 1.5, 1.5))
        wl["src"] = pos
    nsrc = -(-COLUMNS // (((n[0] + 5) // 8) * ((n[1] + 5) // 8)))
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    s, xi, eta, src = (t(wl[k]) for k in ("s", "xi", "eta", "src"))
    src = src.repeat(-(-nsrc // 4), 1)[:nsrc].contiguous()
    assert float(xi.abs().max()) > 0 and float(eta.abs().max()) > 0
    return g, s, xi, eta, src, api.source_params(g, s, xi, eta, src), wl["kappa"], nsrc


def _equal(torch, tau, st, ref, sr, nsrc):
    assert (sr > 0).all()
    for q in (*range(4), nsrc // 2, nsrc - 1):
        assert int(st[q]) == int(sr[q % 4]) and torch.equal(tau[q], ref[q % 4]), q


@pytest.mark.parametrize("coord,n", [(0, (10, 10, 4)), (0, (10, 7, 16)), (0, (11, 19, 31)), (0, (18, 10, 33)),
                                     (0, (20, 27, 50)), (1, (20, 27, 33))])
@pytest.mark.parametrize("mode", ["polled", "asynchronous", "graph"])
def test_lines_modes(torch_cuda, coord, n, mode):
    torch = torch_cuda
    g, s, xi, eta, src, par, kap, nsrc = _problem(torch, coord, n, sum(n))
    assert api.solve_form(g, nsrc, 0)["lines"]
    ref, sr = api.forward(g, s, xi, eta, src[:4].contiguous(), par[:4].contiguous(), 1e-8, 400, kap, poll=True, tile_k=5)
    kw = dict(polled=dict(poll=True), asynchronous={}, graph=dict(graph=True))[mode]
    budget = 400 if mode == "polled" else int(sr.max()) + 3
    for _ in range(2):
        tau, st = api.forward(g, s, xi, eta, src, par, 1e-8, budget, kap, **kw)
        _equal(torch, tau, st, ref, sr, nsrc)


def test_lines_in_a_callers_graph(torch_cuda):
    """Two groups, forked off the captured stream and joined after each has unpadded
    its sources; replayed with another model each time."""
    torch = torch_cuda
    n = (20, 27, 50)
    g, s, xi, eta, src, par, kap, nsrc = _problem(torch, 1, n, 77)
    assert api.solve_form(g, nsrc, 0) == dict(tile_k=16, groups=2, lines=True)
    ws = api.workspace(g, nsrc, 0, device="cuda")
    tau = torch.empty((nsrc,) + n, dtype=torch.float64, device="cuda")
    st = torch.empty(nsrc, dtype=torch.int32, device="cuda")
    budget, model = 40, s.clone()
    run = lambda: api.forward(g, s, xi, eta, src, par, 1e-8, budget, kap, ws=ws, out=tau, status=st)
    run()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    stream = torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=stream):
        run()
    for scale in (1.0, 1.1, 0.9, 1.0):
        s.copy_(model * scale)
        par.copy_(api.source_params(g, s, xi, eta, src))
        tau.zero_()
        graph.replay()
        torch.cuda.synchronize()
        got, gst = tau.clone(), st.clone()
        ref, sr = api.forward(g, s, xi, eta, src[:4].contiguous(), par[:4].contiguous(), 1e-8, budget, kap, poll=True,
                              tile_k=5)
        _equal(torch, got, gst, ref, sr, nsrc)
