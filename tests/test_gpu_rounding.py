"""Rounding of the forward update and of the kernels against the same formulas in
extended precision (NumPy's long double), from the equator to the highest
latitudes that a grid may have.

Forward: a sweep's updates are averages, so rounding errors that are not biased
stay near one unit of the last place.  In Cartesian coordinates, where positions
are exact, the rms error is held to 4e-16, four rms errors of a single rounding at
1; on the sphere the distance to the source is a difference of numbers near 6371
rounded to 5e-13, which near the source is some 1e-15 of tau.

Kernels: the position differences take one rounding of each product kept over the
sources (r cos theta) and none of r sin theta; a float64 evaluation with just
these roundings bounds the error to 5 per cent."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
L = np.longdouble
HAVE_EXTENDED = np.finfo(L).nmant >= 63
needs_extended = pytest.mark.skipif(not HAVE_EXTENDED, reason="long double is no wider than double here")


def _grid(coord, lat_deg, n):
    if coord == 0:
        return dict(n=n, coord=0, o=(0.0, 0.0, 0.0), h=(1.0, 1.0, 1.0))
    h = 2.0 / 6371.0
    hb = h / max(np.cos(np.deg2rad(lat_deg)), 0.05)
    return dict(n=n, coord=1, o=(6371.0 - (n[0] - 1.0), np.deg2rad(lat_deg) - 0.5 * h * (n[1] - 1), -0.5 * hb * (n[2] - 1)),
                h=(1.0, h, hb))


def _inputs(torch, coord, lat_deg, n, nsrc, seed):
    from paper_2412_00031_amd import api
    rng = np.random.default_rng(seed)
    g = _grid(coord, lat_deg, n)
    x = [np.linspace(0.0, 3.0, m) for m in n]
    f = np.cos(x[0])[:, None, None] * np.sin(2 * x[1] + 1)[None, :, None] * np.cos(x[2] + 0.5)[None, None, :]
    s, xi, eta = 0.16 * (1 + 0.15 * f), 0.03 * f * coord, -0.02 * f * coord
    src = np.stack([g["o"][a] + g["h"][a] * (n[a] - 1) * rng.uniform(0.2, 0.8, nsrc) for a in range(3)], 1)
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    d = [t(v) for v in (s, xi, eta, src)]
    par = api.source_params(g, *d)
    ax = [t(g["o"][a] + np.arange(n[a]) * g["h"][a]) for a in range(3)]
    tab = {k: v.cpu().numpy() for k, v in dict(c1=torch.cos(ax[1]), s1=torch.sin(ax[1]), c2=torch.cos(ax[2]),
                                               s2=torch.sin(ax[2])).items()}
    tab["x"] = [a.cpu().numpy() for a in ax]
    # the sources' sines and cosines as the GPU rounds them, like the tables
    tab["src"] = torch.stack([torch.cos(d[3][:, 1]), torch.sin(d[3][:, 1]), torch.cos(d[3][:, 2]),
                              torch.sin(d[3][:, 2])], 1).cpu().numpy()
    return g, (s, xi, eta, src), d, par, tab


def _frame(g, p, trig):
    """Source-frame rows and position, as long doubles."""
    if g["coord"] == 0:
        return np.eye(3, dtype=L), p.astype(L)
    ct, st, cp, sp = (L(v) for v in trig)
    E = np.array([[ct * cp, ct * sp, st], [-st * cp, -st * sp, ct], [-sp, cp, L(0)]])
    return E, L(p[0]) * E[0]


def _minv(par):
    s0, x0, e0 = (L(v) for v in par)
    b, c, f = 1 - 2 * x0, 1 + 2 * x0, 2 * e0
    det = b * c - f * f
    return s0, c / det, -f / det, b / det


def _corner(g, p):
    return [int(np.clip(np.floor((p[a] - g["o"][a]) / g["h"][a]), 0, g["n"][a] - 2)) for a in range(3)]


def _sweeps(g, s, xi, eta, p, trig, par, tab, kappa, iters):
    """Gauss-Seidel sweeps from tau = 1 in extended precision."""
    n, co = g["n"], g["coord"]
    E, Xs = _frame(g, p, trig)
    s0, i11, i12, i22 = _minv(par)
    fb = _corner(g, p)
    h = [L(v) for v in g["h"]]
    fixed = lambda q: all(0 <= q[a] - fb[a] <= 1 for a in range(3))
    f = np.ones(n, dtype=L)
    kappa = L(kappa)
    node = {}
    for i in range(1, n[0] - 1):
        for j in range(1, n[1] - 1):
            for k in range(1, n[2] - 1):
                if fixed((i, j, k)):
                    continue
                x0, x1, x2 = L(tab["x"][0][i]), L(tab["x"][1][j]), L(tab["x"][2][k])
                if co:
                    c1, s1, c2, s2 = (L(tab[q][w]) for q, w in (("c1", j), ("s1", j), ("c2", k), ("s2", k)))
                    D = np.array([x0 * c1 * c2, x0 * c1 * s2, x0 * s1]) - Xs
                else:
                    D = np.array([x0, x1, x2]) - Xs
                d = E @ D
                m = np.array([d[0], i11 * d[1] + i12 * d[2], i12 * d[1] + i22 * d[2]])
                Q = d @ m
                if co:
                    G = m @ E
                    hz = G[0] * c2 + G[1] * s2
                    u = (c1 * hz + s1 * G[2], c1 * G[2] - s1 * hz, G[1] * c2 - G[0] * s2)
                    ga = (L(1), 1 / x0, 1 / (x0 * c1))
                else:
                    u, ga = m, (L(1),) * 3
                C = sum(ga[a] / h[a] for a in range(3))
                node[i, j, k] = (Q, u, [ga[a] / (2 * h[a]) for a in range(3)], s0 / np.sqrt(Q), C,
                                 1 - 2 * L(xi[i, j, k]), 2 * L(eta[i, j, k]), 1 + 2 * L(xi[i, j, k]))
    for _ in range(iters):
        for dr in range(8):
            order = [range(1, n[a] - 1) if not dr >> (2 - a) & 1 else range(n[a] - 2, 0, -1) for a in range(3)]
            for i in order[0]:
                for j in order[1]:
                    for k in order[2]:
                        if (i, j, k) not in node:
                            continue
                        Q, u, v, t, C, ma, mb, mc = node[i, j, k]
                        nb = ((f[i - 1, j, k], f[i + 1, j, k]), (f[i, j - 1, k], f[i, j + 1, k]),
                              (f[i, j, k - 1], f[i, j, k + 1]))
                        R = [Q * ((b - a) * w) + f[i, j, k] * uu for (a, b), w, uu in zip(nb, v, u)]
                        H = t * np.sqrt(R[0] ** 2 + R[1] * (ma * R[1] + mb * R[2]) + R[2] * (mb * R[1] + mc * R[2]))
                        f[i, j, k] = (L(s[i, j, k]) - H) * t / (kappa * s0 * s0 * C) + sum(
                            w / C * (a + b) for (a, b), w in zip(nb, v))
            old = f.copy()
            for q in np.ndindex(n):
                r = list(q)
                while not fixed(r):
                    on = [a for a in range(3) if r[a] in (0, n[a] - 1)]
                    if not on:
                        break
                    r[on[-1]] += 1 if r[on[-1]] == 0 else -1
                f[q] = old[tuple(r)]
    return f


@needs_extended
@pytest.mark.parametrize("coord,lat,bound", [(0, 0.0, 4e-16), (1, 0.0, 2e-15), (1, 45.0, 2e-15), (1, 86.0, 2e-15),
                                             (1, 88.8, 2e-15)])
def test_forward_rounding(torch_cuda, coord, lat, bound):
    from paper_2412_00031_amd import api
    n, nsrc = ((10, 9, 11), 2) if coord else ((14, 13, 15), 1)
    g, (s, xi, eta, src), d, par, tab = _inputs(torch_cuda, coord, lat, n, nsrc, 5)
    kappa = 1.05 if coord else 1.0
    tau, _ = api.forward(g, d[0], d[1], d[2], d[3], par, 1e-300, 8, kappa, poll=True)
    tau, parh = tau.cpu().numpy(), par.cpu().numpy()
    for q in range(nsrc):
        ref = _sweeps(g, s, xi, eta, src[q], tab["src"][q], parh[q], tab, kappa, 8)
        err = float(np.sqrt(np.mean(((tau[q] - ref) / ref) ** 2)))
        assert err <= bound, err


def _kernels(g, xi, eta, src, par, tab, tau, lam, dtype):
    """Kernels of Eqs. (6)-(8); dtype: of all arithmetic past the position differences."""
    n, I = g["n"], (slice(1, -1),) * 3
    T = lambda v: np.asarray(v, dtype=dtype)
    x0, c1, s1, c2, s2 = (T(tab["x"][0])[:, None, None], T(tab["c1"])[None, :, None], T(tab["s1"])[None, :, None],
                          T(tab["c2"])[None, None, :], T(tab["s2"])[None, None, :])
    rct = (x0 * c1).astype(L)  # (rounded to dtype)
    out = np.zeros((3,) + n, dtype=dtype)
    for q in range(len(src)):
        E = T(_frame(g, src[q], tab["src"][q])[0])
        Xs = (T(src[q][0]) * E[0]).astype(L)  # (from the rounded rows, as the library sets it up)
        D = [T(rct * c2.astype(L) - Xs[0]), T(rct * s2.astype(L) - Xs[1]),
             T(x0.astype(L) * s1.astype(L) - Xs[2] + 0 * c2.astype(L))]
        d = [E[i, 0] * D[0] + E[i, 1] * D[1] + E[i, 2] * D[2] for i in range(3)]
        s0, i11, i12, i22 = (T(v) for v in _minv(par[q]))
        m = [d[0], i11 * d[1] + i12 * d[2], i12 * d[1] + i22 * d[2]]
        Q = d[0] * m[0] + d[1] * m[1] + d[2] * m[2]
        f = s0 / np.sqrt(Q)
        G = [f * (m[0] * E[0, a] + m[1] * E[1, a] + m[2] * E[2, a]) for a in range(3)]
        hz = G[0] * c2 + G[1] * s2
        t = [c1 * hz + s1 * G[2], c1 * G[2] - s1 * hz, G[1] * c2 - G[0] * s2]
        P, F = [], T(tau[q])
        for a in range(3):
            hi, lo = [slice(1, -1)] * 3, [slice(1, -1)] * 3
            hi[a], lo[a] = slice(2, None), slice(None, -2)
            w = (F[tuple(hi)] - F[tuple(lo)]) / (2 * T(g["h"][a]))
            if a > 0:
                w = w / (x0 if a == 1 else x0 * c1)[1:-1, slice(None) if a == 1 else slice(1, -1)]
            P.append((f * Q)[I] * w + F[I] * t[a][I])
        X, Y = T(xi)[I], T(eta)[I]
        H = np.sqrt(P[0] ** 2 + P[1] * ((1 - 2 * X) * P[1] + 2 * Y * P[2]) + P[2] * (2 * Y * P[1] + (1 + 2 * X) * P[2]))
        fb = _corner(g, src[q])
        ok = np.ones(n, dtype=bool)
        ok[tuple(slice(b, b + 2) for b in fb)] = False
        lm = np.where(ok, T(lam[q]), 0)[I]
        for c, v in enumerate((1 + 0 * H, (P[1] ** 2 - P[2] ** 2) / H, -2 * P[1] * P[2] / H)):
            out[c][I] += np.where(lm != 0, lm * v, 0)
    return out


@needs_extended
@pytest.mark.parametrize("lat", [0.0, 45.0, 88.0])
def test_kernel_rounding(torch_cuda, lat):
    from paper_2412_00031_amd import api
    torch = torch_cuda
    n = (22, 21, 23)
    g, (s, xi, eta, src), d, par, tab = _inputs(torch, 1, lat, n, 8, 3)
    rng = np.random.default_rng(9)
    tau = np.ones((8,) + n) + 0.05 * np.sin(np.arange(8.0)[:, None, None, None] + np.linspace(0, 4, n[0])[None, :, None, None]
                                            + np.linspace(0, 3, n[1])[None, None, :, None] + np.linspace(0, 5, n[2]))
    lam = rng.standard_normal((8,) + n)
    t = lambda a: torch.as_tensor(a, dtype=torch.float64, device="cuda")
    got = api.kernel(g, d[0], d[1], d[2], d[3], par, t(tau), t(lam)).cpu().numpy()
    parh = par.cpu().numpy()
    ref = _kernels(g, xi, eta, src, parh, tab, tau, lam, L)
    plain = _kernels(g, xi, eta, src, parh, tab, tau, lam, np.float64)
    for c in (1, 2):
        err = float(np.linalg.norm((got[c] - ref[c]).ravel().astype(np.float64)))
        own = float(np.linalg.norm((plain[c] - ref[c]).ravel().astype(np.float64)))
        assert err <= 1.05 * own, (c, err, own)
