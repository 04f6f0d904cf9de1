"""Rounding of the spherical forward update with the source's position kept to more than a
double: distances from the source then round at their own size, not at the Earth's
radius (5e-13), and the error is held to the bound of Cartesian coordinates, four rms
errors of a single rounding at 1, at every latitude and away from longitude 0."""
import numpy as np
import pytest

from test_gpu_rounding import _grid, _sweeps, needs_extended

pytestmark = pytest.mark.gpu


@needs_extended
@pytest.mark.parametrize("lat,lon", [(0.0, 0.0), (45.0, 0.0), (45.0, 118.0), (86.0, 0.0), (-80.0, -60.0), (88.8, 170.0)])
def test_spherical_rounding(torch_cuda, lat, lon):
    torch = torch_cuda
    from paper_2412_00031_amd import api
    n, nsrc, seed = (10, 9, 11), 2, 11
    g = _grid(1, lat, n)
    g["o"] = (g["o"][0], g["o"][1], g["o"][2] + np.deg2rad(lon))
    rng = np.random.default_rng(seed)
    x = [np.linspace(0.0, 3.0, m) for m in n]
    f = np.cos(x[0])[:, None, None] * np.sin(2 * x[1] + 1)[None, :, None] * np.cos(x[2] + 0.5)[None, None, :]
    s, xi, eta = 0.16 * (1 + 0.15 * f), 0.03 * f, -0.02 * f
    src = np.stack([g["o"][a] + g["h"][a] * (n[a] - 1) * rng.uniform(0.2, 0.8, nsrc) for a in range(3)], 1)
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    d = [t(v) for v in (s, xi, eta, src)]
    par = api.source_params(g, *d)
    # node k of an axis lies at o + k h, rounded once as in the tables
    ax = [np.array([float(np.longdouble(g["o"][a]) + np.longdouble(k) * np.longdouble(g["h"][a])) for k in range(n[a])])
          for a in range(3)]
    tab = {k: fn(t(v)).cpu().numpy() for k, fn, v in (("c1", torch.cos, ax[1]), ("s1", torch.sin, ax[1]),
                                                      ("c2", torch.cos, ax[2]), ("s2", torch.sin, ax[2]))}
    tab["x"] = ax
    trig = torch.stack([torch.cos(d[3][:, 1]), torch.sin(d[3][:, 1]), torch.cos(d[3][:, 2]), torch.sin(d[3][:, 2])], 1)
    trig = trig.cpu().numpy()
    tau = api.forward(g, d[0], d[1], d[2], d[3], par, 1e-300, 8, 1.05, poll=True)[0].cpu().numpy()
    parh = par.cpu().numpy()
    for q in range(nsrc):
        ref = _sweeps(g, s, xi, eta, src[q], trig[q], parh[q], tab, 1.05, 8)
        err = float(np.sqrt(np.mean(((tau[q] - ref) / ref) ** 2)))
        print(lat, lon, q, err)
        assert err <= 4e-16, err
