"""Weight gradients where an activation or a gradient has overflowed: an infinite value
reaches the taps whose products it is in and no others.  (A row's last input is not
an input of the tap dx = -1; a gradient in the first plane meets no input of dz =
-1, one in the last row none of dy = 1.)"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _wgrad(x, g):
    """Products inside the volume only, tap by tap."""
    D, H, W = x.shape[:3]
    out = np.zeros((27, x.shape[3], g.shape[3]))
    with np.errstate(invalid="ignore"):
        for t in range(27):
            d = (t // 9 - 1, t // 3 % 3 - 1, t % 3 - 1)
            lo = [max(0, -v) for v in d]
            hi = [n - max(0, v) for n, v in zip((D, H, W), d)]
            xs = x[tuple(slice(a + v, b + v) for a, b, v in zip(lo, hi, d))]
            gs = g[tuple(slice(a, b) for a, b in zip(lo, hi))]
            out[t] = (xs[..., :, None] * gs[..., None, :]).sum((0, 1, 2))
    return out


@pytest.mark.parametrize("dims", [(3, 4, 5), (2, 3, 33), (2, 2, 64), (3, 3, 70)])
@pytest.mark.parametrize("where", ["input at a row's end", "gradient in the first plane", "gradient in the last row"])
@pytest.mark.parametrize("cin,cout", [(16, 16), (32, 32)])
def test_conv3_wgrad_infinite(torch_cuda, dims, where, cin, cout):
    from paper_2412_00031_amd import nn
    torch = torch_cuda
    rng = np.random.default_rng(dims[2])
    D, H, W = dims
    bf = lambda a: torch.as_tensor(a.astype(np.float32)).to(torch.bfloat16)
    x, g = rng.uniform(0.5, 1.5, dims + (cin,)), rng.uniform(0.5, 1.5, dims + (cout,))
    if where == "input at a row's end":
        x[1, 1, W - 1, 3] = np.inf
    elif where == "gradient in the first plane":
        g[0, H // 2, W // 2, 5] = np.inf
    else:
        g[D - 1, H - 1, W // 2, 5] = -np.inf
    xb, gb = bf(x), bf(g)
    gW, _ = nn.conv3_wgrad(xb[None].cuda(), cin, gb[None].cuda(), cout)
    got, ref = gW.double().cpu().numpy(), _wgrad(xb.double().numpy(), gb.double().numpy())
    fin = np.isfinite(ref)
    assert fin.any() and not fin.all()
    assert np.array_equal(np.isfinite(got), fin), np.argwhere(np.isfinite(got) != fin)[:5]
    assert np.array_equal(got[~fin], ref[~fin])
    assert np.allclose(got[fin], ref[fin], rtol=1e-5, atol=0)
