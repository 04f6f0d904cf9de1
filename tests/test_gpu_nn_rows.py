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


# Tiles of a plane at their edges: one row, ragged last tiles, rows of one
# 16-position block and a rest, rows as wide as a tile, every count of channel
# blocks, z chunks; and the layouts that go to the direct kernel (48 input
# channels, rows wider than a tile, odd channel offsets).
@pytest.mark.parametrize("cin,cout,nb,dims,offs", [
    (16, 16, 1, (1, 1, 1), (0, 0)), (16, 16, 2, (9, 19, 56), (8, 4)), (16, 32, 1, (8, 12, 33), (0, 0)),
    (16, 48, 1, (3, 7, 17), (8, 0)), (16, 64, 1, (2, 30, 9), (0, 8)), (32, 16, 1, (5, 23, 56), (0, 0)),
    (32, 32, 2, (4, 28, 28), (16, 0)), (64, 32, 1, (6, 14, 14), (0, 4)), (64, 64, 1, (7, 7, 7), (0, 0)),
    (16, 16, 1, (2, 2, 512), (0, 0)), (16, 16, 1, (2, 2, 513), (0, 0)), (48, 16, 1, (3, 5, 20), (0, 0)),
    (32, 16, 1, (3, 5, 20), (4, 0)), (16, 16, 1, (3, 5, 20), (0, 3))])
def test_conv3_planes(torch_cuda, cin, cout, nb, dims, offs):
    from paper_2412_00031_amd import nn
    torch = torch_cuda
    rng = np.random.default_rng(cin * 3 + cout + dims[1])
    cxo, cyo = offs
    cxt = cin + 16 if cxo % 8 == 0 else cin + 4
    x_d, x = _bf(torch, rng.standard_normal((nb,) + dims + (cxt,)))
    W = rng.standard_normal((27, cin, cout)) * 0.2
    W_d = torch.as_tensor(W.astype(np.float32)).cuda()
    b = rng.standard_normal(cout).astype(np.float32)
    y_d = torch.full((nb,) + dims + (cout + 12,), 7.0, dtype=torch.bfloat16, device="cuda")
    nn.conv3_fwd(x_d, cin, nn.conv3_pack(W_d), torch.as_tensor(b).cuda(), cout, True, y_d, cx_off=cxo, cy_off=cyo)
    got = y_d.double().cpu().numpy()
    Wr = torch.as_tensor(W.astype(np.float32)).to(torch.bfloat16).double().numpy()
    for q in range(nb):
        xs = x[q, ..., cxo:cxo + cin]
        ref = np.maximum(U.conv3(xs, Wr, b.astype(np.float64)), 0.0)
        mag = U.conv3(np.abs(xs), np.abs(Wr), np.abs(b).astype(np.float64))
        out = got[q, ..., cyo:cyo + cout]
        assert np.all(np.abs(out - ref) <= 2.0 ** -8 * np.abs(ref) + 1e-6 * mag), np.abs(out - ref).max()
        rest = np.delete(got[q], np.s_[cyo:cyo + cout], axis=-1)
        assert np.all(rest == 7.0)
