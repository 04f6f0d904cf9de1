"""Host logic of how a solve runs: the default form of a batch, what explicit options
make of it, workspaces that were sized for other options, and the tuner's choice
between the default and explicit depths."""
import ctypes
import os

import pytest


@pytest.fixture(scope="module")
def api():
    from paper_2412_00031_amd import _lib, api, build
    if not os.path.exists(_lib.LIB_PATH):
        build.build()
    _lib.load(_lib.LIB_PATH)
    return api


def _size(api, g, nsrc, which, **kw):
    from paper_2412_00031_amd import _lib
    o = api._opts(1e-6, 1, 1.0, kw.get("tile_k", 0), groups=kw.get("groups", 0), compact=kw.get("compact", False))
    return _lib.load().tt_workspace_size(ctypes.byref(api._grid(g)), nsrc, ctypes.byref(o), which)


def _grid(n):
    return dict(n=(n, n, n), coord=1, o=(6371.0 - (n - 1), -0.01, -0.01), h=(1.0, 0.02 / (n - 1), 0.02 / (n - 1)))


def test_default_form_by_batch(api):
    assert api.solve_form(_grid(41), 1, 0) == dict(tile_k=16, groups=1, lines=False)
    assert api.solve_form(_grid(61), 64, 0) == dict(tile_k=16, groups=2, lines=True)
    assert api.solve_form(_grid(101), 128, 0) == dict(tile_k=28, groups=1, lines=False)
    assert api.solve_form(_grid(101), 128, 1) == dict(tile_k=40, groups=2, lines=False)
    assert api.solve_form(_grid(61), 64, 0, tile_k=20) == dict(tile_k=20, groups=1, lines=False)
    assert api.solve_form(_grid(61), 64, 0, time_sweeps=True)["groups"] == 1
    with pytest.raises(RuntimeError):
        api.solve_form(_grid(61), 64, 0, tile_k=63)


def test_workspace_of_an_explicit_depth_has_no_padded_fields(api):
    g, nsrc = _grid(61), 64
    fields = 8 * nsrc * 61 ** 3
    assert _size(api, g, nsrc, 0) > fields
    assert _size(api, g, nsrc, 0, tile_k=28) < _size(api, g, nsrc, 0) - fields
    # the default then solves in place on it
    assert not api.solve_form(g, nsrc, 0, ws_bytes=_size(api, g, nsrc, 0, tile_k=28))["lines"]


@pytest.mark.parametrize("which", [0, 1])
def test_workspace_sized_for_other_groups_serves(api, which):
    for n, nsrc in ((61, 64), (41, 100), (101, 128), (21, 16)):
        g = _grid(n)
        for sized in (0, 1, 2):
            have = _size(api, g, nsrc, which, groups=sized)
            for asked in (1, 2, 4, 8):
                f = api.solve_form(g, nsrc, which, groups=asked, ws_bytes=have)
                assert 1 <= f["groups"] <= asked
                # what it settles on fits, in place or padded
                if not f["lines"]:
                    assert _size(api, g, nsrc, which, groups=f["groups"], tile_k=f["tile_k"]) <= have
        full = _size(api, g, nsrc, which, groups=4)
        assert api.solve_form(g, nsrc, which, groups=4, ws_bytes=full)["groups"] == 4


def test_tuner_can_choose_the_default_form(api, monkeypatch):
    import torch
    from paper_2412_00031_amd import autotune
    g, nsrc = _grid(21), 8
    asked = []

    def timed(kind, grid, s, xi, eta, src, par, tau, rec, R, kappa, tk, groups, iters):
        asked.append((kind, tk, groups))
        return 1.0 if (tk, groups) == (0, 0) else 2.0

    monkeypatch.setattr(autotune, "_time", timed)
    monkeypatch.setattr(autotune.api, "forward", lambda *a, **k: (torch.zeros(nsrc, 1), None))
    z = torch.zeros(1, dtype=torch.float64)
    got = autotune.tune(g, z, z, z, torch.zeros(nsrc, 3), torch.zeros(nsrc, 3), 1.05, torch.zeros(2, 3), use_cache=False)
    assert got == {"fwd": 0, "adj": 0, "groups_fwd": 0, "groups_adj": 0, "cached": False}
    assert ("fwd", 16, 0) in asked and ("adj", 0, 2) in asked


@pytest.mark.parametrize("n,nsrc", [(101, 3), (61, 20), (41, 8)])
def test_adjoint_workspace_holds_what_both_systems_use(api, n, nsrc):
    """Records, diagonal, right-hand side and two values per boundary node and source;
    nothing that only the continuous system needs."""
    N, NB = n ** 3, n ** 3 - (n - 2) ** 3
    per_source = 8 * (2 * N + 2 * NB)
    full = 4 * n * (2 * n - 1) * ((n + 14) // 8 * 8) * 48
    slack = 64 * 1024 + nsrc * 8 * NB  # tables, sums and progress words
    assert _size(api, _grid(n), nsrc, 1, groups=1) <= nsrc * (per_source + full) + slack
    assert _size(api, _grid(n), nsrc, 1, groups=1, compact=True) <= nsrc * (per_source + 48 * N) + slack
