"""Common-receiver misfit with observed clock times: T_obs is some 1.7e9 s, whose last
place is 2.4e-7 s, so differences have to be taken source against source before
T meets T_obs.  Oracle and kernel then form the same residuals and only the sum's
order differs: eps times the number of terms."""
import numpy as np
import pytest

import oracle as O
from paper_2412_00031_amd import api

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -52


# receivers staged in one run, in several, and more sources than a run holds
@pytest.mark.parametrize("nsrc,nrec", [(4, 30), (30, 700), (9601, 3)])
def test_misfit_cr_clock_times(torch_cuda, nsrc, nrec):
    torch = torch_cuda
    rng = np.random.default_rng(nsrc)
    T = rng.uniform(1, 20, (nsrc, nrec))
    Tobs = 1.7e9 + T + rng.normal(0, 0.2, T.shape)
    cnt = rng.integers(0, 20, nrec)
    off = np.concatenate([[0], np.cumsum(cnt)]).astype(np.int32)
    pair = rng.integers(0, nsrc, (off[-1], 2)).astype(np.int32)
    tri = np.concatenate([pair, np.repeat(np.arange(nrec), cnt)[:, None]], 1).astype(np.int32)
    chi_o, _ = O.misfit_cr(T, Tobs, tri, np.ones(len(pair)), 0.9)
    d = lambda a, dt=torch.float64: torch.as_tensor(np.ascontiguousarray(a), dtype=dt, device="cuda")
    chi, R = torch.zeros((), dtype=torch.float64, device="cuda"), torch.zeros((nsrc, nrec), dtype=torch.float64, device="cuda")
    api.misfit_cr(d(T), d(Tobs), d(off, torch.int32), d(pair, torch.int32), None, 0.9, R, chi)
    assert abs(chi.item() - chi_o) <= (len(pair) + 4) * EPS * chi_o
