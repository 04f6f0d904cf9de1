"""Default form of an adjoint solve over batch sizes: the depth of its slabs and its
source groups at the edges of their rules, and odd source counts."""
import os

import pytest


@pytest.fixture(scope="module")
def form():
    from paper_2412_00031_amd import _lib, api, build
    if not os.path.exists(_lib.LIB_PATH):
        build.build()
    _lib.load(_lib.LIB_PATH)

    def f(n, nsrc, **kw):
        g = dict(n=n, coord=0, o=(0.0, 0.0, 0.0), h=(1.0, 1.0, 1.0))
        r = api.solve_form(g, nsrc, 1, **kw)
        return r["tile_k"], r["groups"]

    return f


@pytest.mark.parametrize("n,nsrc,want", [
    ((41, 41, 41), 1, (16, 1)),
    ((61, 61, 61), 8, (16, 1)), ((61, 61, 61), 9, (16, 2)), ((61, 61, 61), 16, (16, 2)),
    ((61, 61, 61), 17, (16, 3)), ((61, 61, 61), 32, (16, 4)), ((61, 61, 61), 33, (40, 3)),
    ((101, 101, 101), 8, (16, 1)), ((101, 101, 101), 9, (40, 2)), ((101, 101, 101), 18, (40, 3)),
    ((101, 101, 101), 40, (40, 3)), ((101, 101, 101), 128, (40, 2)),
    ((33, 25, 82), 34, (16, 1)), ((33, 25, 82), 255, (40, 3)),
    ((101, 101, 25), 12, (16, 2)), ((101, 101, 25), 24, (40, 3)),  # columns alone
])
def test_adjoint_form_by_batch(form, n, nsrc, want):
    """A batch leaves the shallow slabs when its nodes and not its columns outgrow them,
    and has a group for every eight sources begun."""
    assert form(n, nsrc) == want


def test_explicit_options_stand(form):
    assert form((101, 101, 101), 18, tile_k=16) == (16, 3)
    assert form((101, 101, 101), 18, groups=5) == (40, 5)
    assert form((61, 61, 61), 3, groups=8) == (16, 3)
    assert form((101, 101, 101), 18, time_sweeps=True) == (40, 1)
