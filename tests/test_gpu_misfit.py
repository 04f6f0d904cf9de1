"""The misfit's blocks take receivers and pairs in chunks: chi and R against the
oracle at the chunks' edges.  R's elements receive the oracle's additions in the
oracle's order, so that only the contraction of multiply-adds differs: n
additions round n times, eps each of the terms' sum.  chi sums the same positive
terms in another order: eps times their number."""
import numpy as np
import pytest

import oracle as O
from paper_2412_00031_amd import api

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -52


# pairs: none, one, a chunk (1024) and one more, many at one receiver (a star,
# walked instead of sorted); receivers past one listing (4096); one source, past
# one block's sources (256)
@pytest.mark.parametrize("nsrc,nrec,npair,star", [(1, 1, 0, False), (1, 2, 1, False), (3, 40, 1024, False),
                                                  (2, 700, 1025, True), (257, 9, 36, False), (2, 4100, 3000, False),
                                                  (2, 64, 33, True), (2, 64, 32, True)])
def test_misfit_chunks(torch_cuda, nsrc, nrec, npair, star):
    torch = torch_cuda
    rng = np.random.default_rng(nsrc * 1000 + nrec)
    T = rng.uniform(1, 20, (nsrc, nrec))
    Tobs = T + rng.normal(0, 0.2, T.shape)
    w = rng.uniform(0.5, 1.5, T.shape)
    pairs = rng.integers(0, nrec, (npair, 2)).astype(np.int32)
    if star:
        pairs[:, npair % 2] = nrec // 2
    wp = rng.uniform(0.5, 2.0, (nsrc, npair))
    chi_o, R_o = O.misfit(T, Tobs, w, pairs, wp, alpha=0.7, beta=1.3)
    d = lambda a, dt=torch.float64: torch.as_tensor(np.ascontiguousarray(a), dtype=dt, device="cuda")
    chi, R = api.misfit(d(T), d(Tobs), d(w), d(pairs, torch.int32) if npair else None, d(wp) if npair else None, 0.7, 1.3)
    size = np.abs(0.7 * w * (T - Tobs))
    n = np.ones(T.shape)
    for p, (a, b) in enumerate(pairs):
        t = np.abs(1.3 * wp[:, p] * ((T[:, a] - T[:, b]) - (Tobs[:, a] - Tobs[:, b])))
        for m in (a, b):
            size[:, m] += t
            n[:, m] += 1
    # three roundings within a term, one per addition; differences of T are the same on both sides
    assert (np.abs(R.cpu().numpy() - R_o) <= (n + 3) * EPS * size).all()
    assert abs(chi.item() - chi_o) <= (nsrc * (nrec + npair) + 4) * EPS * chi_o


# sources per run of receivers: one receiver a run (more than 7168 sources), a
# partial last run, and more sources than the residuals in LDS
@pytest.mark.parametrize("nsrc,nrec", [(2, 600), (30, 500), (7200, 3), (14337, 2)])
def test_misfit_cr_runs(torch_cuda, nsrc, nrec):
    torch = torch_cuda
    rng = np.random.default_rng(nsrc + nrec)
    T = rng.uniform(1, 20, (nsrc, nrec))
    Tobs = T + rng.normal(0, 0.2, T.shape)
    cnt = rng.integers(0, 90, nrec)  # past one stage of 64 pairs
    off = np.concatenate([[0], np.cumsum(cnt)]).astype(np.int32)
    pair = rng.integers(0, nsrc, (off[-1], 2)).astype(np.int32)
    tri = np.concatenate([pair, np.repeat(np.arange(nrec), cnt)[:, None]], 1).astype(np.int32)
    wc = rng.uniform(0.5, 2.0, len(pair))
    chi_o, R_o = O.misfit_cr(T, Tobs, tri, wc, 0.9)
    d = lambda a, dt=torch.float64: torch.as_tensor(np.ascontiguousarray(a), dtype=dt, device="cuda")
    chi, R = torch.zeros((), dtype=torch.float64, device="cuda"), torch.zeros((nsrc, nrec), dtype=torch.float64, device="cuda")
    api.misfit_cr(d(T), d(Tobs), d(off, torch.int32), d(pair, torch.int32), d(wc), 0.9, R, chi)
    size, n = np.zeros(T.shape), np.zeros(T.shape)
    for p, (a, b, m) in enumerate(tri):
        t = abs(0.9 * wc[p] * ((T[a, m] - T[b, m]) - (Tobs[a, m] - Tobs[b, m])))
        for q in (a, b):
            size[q, m] += t
            n[q, m] += 1
    assert (np.abs(R.cpu().numpy() - R_o) <= (n + 3) * EPS * size).all()
    # the kernel takes (T - Tobs) first, the oracle T - T: three roundings of
    # values up to 20.2 each, times gamma w r, the derivative of the term
    dr = 6 * EPS * 20.2 * size.sum()
    assert abs(chi.item() - chi_o) <= (len(pair) + 4) * EPS * chi_o + dr
