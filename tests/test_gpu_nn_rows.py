"""Weight gradients from LDS-staged rows: row lengths around the 32-position
matrix steps and the 64-position chunks, several rows per slice, channel blocks
of every instance, against the float64 NumPy reference.  Sums of n products of
bf16 values in fp32: |error| <= n 2^-24 max|x| max|g| at worst, far less in
practice; the bound below is 1e-5 of the sum of absolute products."""
import numpy as np
import pytest

from oracle import unet_ref as U

pytestmark = pytest.mark.gpu


def _bf(torch, a):
    t = torch.as_tensor(np.asarray(a, dtype=np.float32)).to(torch.bfloat16)
    return t.cuda(), t.double().numpy()


def _check(got, ref, mag):
    got = got.double().cpu().numpy()
    assert np.all(np.abs(got - ref) <= 1e-5 * mag + 1e-30), np.max(np.abs(got - ref) / mag)


@pytest.mark.parametrize("cin,cout,dims", [(16, 16, (2, 3, 32)), (4, 32, (3, 9, 33)), (32, 16, (2, 5, 64)),
                                           (64, 32, (2, 4, 65)), (48, 48, (1, 2, 70)), (32, 64, (9, 8, 5)),
                                           (16, 16, (1, 1, 1))])
def test_conv3_wgrad_rows(torch_cuda, cin, cout, dims):
    from paper_2412_00031_amd import nn
    torch = torch_cuda
    rng = np.random.default_rng(cin + cout + dims[2])
    cxt = 16 * ((cin + 15) // 16) + 8
    x_d, x = _bf(torch, rng.standard_normal((2,) + dims + (cxt,)))
    g_d, g = _bf(torch, rng.standard_normal((2,) + dims + (cout + 8,)))
    gW, gb = nn.conv3_wgrad(x_d, cin, g_d, cout, cx_off=0, cg_off=8)
    ref, mag, refb, magb = 0.0, 0.0, 0.0, 0.0
    for q in range(2):
        Z = np.zeros((27, cin, cout))
        _, w, b = U.conv3_backward(x[q, ..., :cin], Z, g[q, ..., 8:])
        _, wm, bm = U.conv3_backward(np.abs(x[q, ..., :cin]), Z, np.abs(g[q, ..., 8:]))
        ref, mag, refb, magb = ref + w, mag + wm, refb + b, magb + bm
    _check(gW, ref, mag)
    _check(gb, refb, magb)
    gW2, none = nn.conv3_wgrad(x_d, cin, g_d, cout, cx_off=0, cg_off=8, with_bias=False)
    assert none is None and torch.equal(gW2, gW)


@pytest.mark.parametrize("cin,cout,dims", [(16, 16, (2, 3, 32)), (32, 16, (1, 9, 33)), (64, 32, (2, 2, 64)),
                                           (48, 32, (1, 2, 65)), (32, 48, (3, 2, 4)), (16, 16, (1, 1, 1))])
def test_up_wgrad_rows(torch_cuda, cin, cout, dims):
    from paper_2412_00031_amd import nn
    torch = torch_cuda
    rng = np.random.default_rng(3 * cin + cout + dims[2])
    x_d, x = _bf(torch, rng.standard_normal((2,) + dims + (cin,)))
    g_d, g = _bf(torch, rng.standard_normal((2,) + tuple(2 * d for d in dims) + (cout + 16,)))
    Wu = rng.standard_normal((8, cin, cout))
    W_d = torch.as_tensor(Wu.astype(np.float32)).cuda()
    _, gW, gb = nn.up_bwd(x_d, g_d, W_d, cg_off=8)
    ref, mag, refb, magb = 0.0, 0.0, 0.0, 0.0
    for q in range(2):
        gq = g[q, ..., 8:8 + cout]
        _, w, b = U.up_backward(x[q], Wu, gq)
        _, wm, bm = U.up_backward(np.abs(x[q]), Wu, np.abs(gq))
        ref, mag, refb, magb = ref + w, mag + wm, refb + b, magb + bm
    _check(gW, ref, mag)
    _check(gb, refb, magb)
