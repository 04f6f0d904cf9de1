"""Host logic of the sliced weight gradients: every slice of rows starts inside
the tensor.  The slice counts are read back from the scratch sizes."""
import os

import pytest


@pytest.fixture(scope="module")
def lib():
    from paper_2412_00031_amd import _lib, build
    if not os.path.exists(_lib.LIB_PATH):
        build.build()
    return _lib.load(_lib.LIB_PATH)


def _rows():
    return sorted(set(range(1, 700)) | set(range(2040, 2060)) | set(range(4090, 4110)) |
                  {5184, 6272, 6400, 10816, 12544, 65537} | {p * p * p // 7 for p in range(20, 200, 3)})


def _starts_inside(nrows, ns):
    rows = -(-nrows // ns)
    return (ns - 1) * rows < nrows


def test_no_empty_weight_gradient_slice(lib):
    per = 4 * (27 * 16 * 16 + 16)
    for nrows in _rows():
        size = lib.nn_conv3_wgrad_work(1, 1, nrows, 1, 16, 16)
        assert size % per == 0
        ns = size // per
        assert 1 <= ns <= 512 and _starts_inside(nrows, ns), (nrows, ns)


def test_no_empty_up_sampling_slice(lib):
    per = 4 * (8 * 16 * 16 + 4 * 16)
    for nrows in _rows():
        # (one position a row: the rows' own scratch is the largest of the three forms')
        size = lib.nn_up_wgrad_work(1, 1, nrows, 1, 16, 16)
        if size % per:
            continue
        ns = size // per
        assert 1 <= ns <= 512 and _starts_inside(nrows, ns), (nrows, ns)
    assert lib.nn_up_wgrad_work(1, 1, 5184, 1, 16, 16) % per == 0
