"""Edges of the rules that give small calls more waves: the weight gradient's slices
(one row up to 32, then rows in eights), the up-sampling's form below and above 512
positions, and the warm start's interpolation in pieces of 64 nodes for fewer than
8 sources.  Bounds as for the general forms."""
import numpy as np
import pytest

from oracle import unet_ref as U

pytestmark = pytest.mark.gpu


def _bf(torch, a):
    t = torch.as_tensor(np.asarray(a, dtype=np.float32)).to(torch.bfloat16)
    return t.cuda(), t.double().numpy()


@pytest.mark.parametrize("dims", [(1, 2, 3), (4, 8, 2), (3, 11, 2), (8, 32, 2), (257, 1, 2)])
def test_wgrad_few_rows(torch_cuda, dims):
    from paper_2412_00031_amd import nn
    torch = torch_cuda
    rng = np.random.default_rng(dims[1])
    x_d, x = _bf(torch, rng.standard_normal((1,) + dims + (16,)))
    g_d, g = _bf(torch, rng.standard_normal((1,) + dims + (16,)))
    gW, gb = nn.conv3_wgrad(x_d, 16, g_d, 16)
    Z = np.zeros((27, 16, 16))
    _, w, b = U.conv3_backward(x[0], Z, g[0])
    _, wm, bm = U.conv3_backward(np.abs(x[0]), Z, np.abs(g[0]))
    for got, ref, mag in ((gW, w, wm), (gb, b, bm)):
        assert np.all(np.abs(got.double().cpu().numpy() - ref) <= 1e-5 * mag + 1e-30)


@pytest.mark.parametrize("nb,dims", [(1, (8, 8, 8)), (1, (27, 19, 1)), (2, (4, 8, 8))])
def test_up_few_positions(torch_cuda, nb, dims):
    from paper_2412_00031_amd import nn
    torch = torch_cuda
    rng = np.random.default_rng(dims[0])
    x_d, x = _bf(torch, rng.standard_normal((nb,) + dims + (32,)))
    Wu, b = rng.standard_normal((8, 32, 16)).astype(np.float32), rng.standard_normal(16).astype(np.float32)
    y_d = torch.empty((nb,) + tuple(2 * d for d in dims) + (16,), dtype=torch.bfloat16, device="cuda")
    nn.up_fwd(x_d, torch.as_tensor(Wu).cuda(), torch.as_tensor(b).cuda(), y_d)
    y = y_d.double().cpu().numpy()
    for q in range(nb):
        ref = U.up(x[q], Wu.astype(np.float64), b.astype(np.float64))
        mag = U.up(np.abs(x[q]), np.abs(Wu).astype(np.float64), np.abs(b).astype(np.float64))
        assert np.all(np.abs(y[q] - ref) <= 2.0 ** -8 * np.abs(ref) + 1e-5 * mag)


# 7 sources in pieces, 8 in runs, from the same predictions: bit for bit
@pytest.mark.parametrize("n", [(5, 6, 64), (6, 5, 65), (12, 9, 200)])
def test_warm_init_pieces(torch_cuda, n):
    from paper_2412_00031_amd import nn
    torch = torch_cuda
    rng = np.random.default_rng(n[2])
    g = dict(n=n, coord=0, o=(0.0, 0.0, 0.0), h=(1.0, 1.0, 1.0))
    dims = tuple((v - 1) // 3 + 2 for v in n)
    pred = torch.as_tensor(rng.standard_normal((8,) + dims).astype(np.float32)).cuda()
    few, many = nn.warm_init(g, pred[:7].contiguous(), 3), nn.warm_init(g, pred, 3)
    N = n[0] * n[1] * n[2]
    assert torch.equal(few.reshape(7, N), many.reshape(8, N)[:7])
