"""Weight gradients over more rows than there are slices, in counts that do not
divide: the slices are then several rows long and the last one is short.  Bounds
as for the staged rows: 1e-5 of the sum of absolute products."""
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


@pytest.mark.parametrize("nb,dims,cin,cout", [(1, (72, 72, 5), 16, 16), (2, (57, 37, 3), 32, 16)])
def test_conv3_wgrad_many_rows(torch_cuda, nb, dims, cin, cout):
    from paper_2412_00031_amd import nn
    torch = torch_cuda
    rng = np.random.default_rng(cin + dims[1])
    x_d, x = _bf(torch, rng.standard_normal((nb,) + dims + (cin,)))
    g_d, g = _bf(torch, rng.standard_normal((nb,) + dims + (cout,)))
    gW, gb = nn.conv3_wgrad(x_d, cin, g_d, cout)
    ref, mag, refb, magb = 0.0, 0.0, 0.0, 0.0
    for q in range(nb):
        Z = np.zeros((27, cin, cout))
        _, w, b = U.conv3_backward(x[q], Z, g[q])
        _, wm, bm = U.conv3_backward(np.abs(x[q]), Z, np.abs(g[q]))
        ref, mag, refb, magb = ref + w, mag + wm, refb + b, magb + bm
    _check(gW, ref, mag)
    _check(gb, refb, magb)


def test_up_wgrad_many_rows(torch_cuda):
    from paper_2412_00031_amd import nn
    torch = torch_cuda
    rng = np.random.default_rng(11)
    dims, cin, cout = (46, 47, 3), 32, 16
    x_d, x = _bf(torch, rng.standard_normal((1,) + dims + (cin,)))
    g_d, g = _bf(torch, rng.standard_normal((1,) + tuple(2 * d for d in dims) + (cout,)))
    Wu = rng.standard_normal((8, cin, cout))
    _, gW, gb = nn.up_bwd(x_d, g_d, torch.as_tensor(Wu.astype(np.float32)).cuda())
    _, w, b = U.up_backward(x[0], Wu, g[0])
    _, wm, bm = U.up_backward(np.abs(x[0]), Wu, np.abs(g[0]))
    _check(gW, w, wm)
    _check(gb, b, bm)
