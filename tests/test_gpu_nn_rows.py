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


# channel counts and offsets that do not come in aligned pieces of 8, beside ones that do
@pytest.mark.parametrize("cin,cout,off", [(16, 16, 8), (5, 3, 1), (24, 16, 4), (64, 32, 16), (8, 48, 0)])
def test_up_head_pool_mask_forms(torch_cuda, cin, cout, off):
    from paper_2412_00031_amd import nn
    torch = torch_cuda
    rng = np.random.default_rng(cin + 5 * cout + off)
    nb, D, H, W = 2, 3, 2, 5
    x_d, x = _bf(torch, rng.standard_normal((nb, D, H, W, cin)))
    Wu = rng.standard_normal((8, cin, cout)).astype(np.float32)
    b = rng.standard_normal(cout).astype(np.float32)
    y_d = torch.full((nb, 2 * D, 2 * H, 2 * W, cout + off + 8), 3.0, dtype=torch.bfloat16, device="cuda")
    W_d, b_d = torch.as_tensor(Wu).cuda(), torch.as_tensor(b).cuda()
    nn.up_fwd(x_d, W_d, b_d, y_d, cy_off=off)
    g_d, g = _bf(torch, rng.standard_normal(tuple(y_d.shape)))
    gx_d, _, _ = nn.up_bwd(x_d, g_d, W_d, cg_off=off)
    y = y_d.double().cpu().numpy()
    for q in range(nb):
        gq = g[q, ..., off:off + cout]
        for got, ref, mag in ((y[q, ..., off:off + cout], U.up(x[q], Wu.astype(np.float64), b.astype(np.float64)),
                               U.up(np.abs(x[q]), np.abs(Wu).astype(np.float64), np.abs(b).astype(np.float64))),
                              (gx_d[q].double().cpu().numpy(), U.up_backward(x[q], Wu.astype(np.float64), gq)[0],
                               U.up_backward(x[q], np.abs(Wu).astype(np.float64), np.abs(gq))[0])):
            assert np.all(np.abs(got - ref) <= 2.0 ** -8 * np.abs(ref) + 1e-5 * mag)
    assert np.all(np.delete(y, np.s_[off:off + cout], axis=-1) == 3.0)
    # head: forward, data and weight gradients
    w = rng.standard_normal(cin).astype(np.float32)
    w_d = torch.as_tensor(w).cuda()
    yh = nn.head_fwd(x_d, w_d, torch.zeros(1, device="cuda"))
    gh = rng.standard_normal((nb, D, H, W)).astype(np.float32)
    gxh, gw, gb = nn.head_bwd(x_d, torch.as_tensor(gh).cuda(), w_d)
    _check(yh, x @ w.astype(np.float64), np.abs(x) @ np.abs(w).astype(np.float64))
    want = torch.as_tensor(gh[..., None] * w).to(torch.bfloat16)
    assert torch.equal(gxh.cpu(), want)
    _check(gw, np.einsum("nzyxi,nzyx->i", x, gh), np.einsum("nzyxi,nzyx->i", np.abs(x), np.abs(gh)))
    _check(gb, np.array([gh.astype(np.float64).sum()]), np.abs(gh).sum())
    # pooling and mask, exact, on channels [off, off + cin) of a wider array of small integers (ties)
    t_d, t = _bf(torch, rng.integers(-2, 3, (nb, 4, 2, 6, cin + off + 8)).astype(np.float64))
    p_d = nn.pool_fwd(t_d, cin, c_off=off)
    gp_d, gp = _bf(torch, rng.standard_normal((nb, 2, 1, 3, cin)))
    gt_d = torch.ones_like(t_d)
    nn.pool_bwd(t_d, gp_d, cin, gt_d, c_off=off, accumulate=True)
    m_d = torch.full((nb, 4, 2, 6, cin + off), 5.0, dtype=torch.bfloat16, device="cuda")
    gm_d, gm = _bf(torch, rng.standard_normal(t.shape))
    nn.relu_mask(gm_d, t_d, cin, m_d, c_off=off, co_off=off)
    for q in range(nb):
        ts = t[q, ..., off:off + cin]
        assert np.array_equal(p_d[q].double().cpu().numpy(), U.pool(ts))
        want = torch.as_tensor(1.0 + U.pool_backward(ts, gp[q])).float().to(torch.bfloat16)
        assert torch.equal(gt_d[q, ..., off:off + cin].cpu(), want)
    assert np.all(np.delete(gt_d.double().cpu().numpy(), np.s_[off:off + cin], axis=-1) == 1.0)
    assert np.array_equal(m_d[..., off:].double().cpu().numpy(), np.where(t > 0, gm, 0.0)[..., off:off + cin])
    assert np.all(m_d[..., :off].double().cpu().numpy() == 5.0)


# rows of the grid longer than a wave, one-node axes of the coarse grid, strides that leave a rest
@pytest.mark.parametrize("n,stride,coord", [((5, 6, 131), 2, 1), ((4, 70, 9), 3, 0), ((9, 8, 65), 1, 1), ((4, 4, 4), 7, 0)])
def test_warm_rows(torch_cuda, n, stride, coord):
    from paper_2412_00031_amd import nn
    torch = torch_cuda
    rng = np.random.default_rng(sum(n) + stride)
    g = dict(n=n, coord=coord, o=(6300.0, -0.02, 0.3), h=(1.0, 3e-4, 4e-4)) if coord else dict(n=n, coord=0, o=(0.0, 1.0, 2.0), h=(1.0, 2.0, 0.5))
    m = tuple((v - 1) // stride + 1 for v in n)
    dims = tuple(v + 2 for v in m)
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    s, xi, eta = rng.uniform(0.1, 0.3, n), rng.uniform(-0.05, 0.05, n), rng.uniform(-0.05, 0.05, n)
    lo = np.array(g["o"])
    src = lo + rng.uniform(0.0, 1.0, (2, 3)) * np.array(g["h"]) * (np.array(n) - 1)
    par = np.stack([[0.2, 0.0, 0.0], [0.15, 0.0, 0.0]])
    f = nn.warm_features(g, t(s), t(xi), t(eta), t(src), t(par), stride, dims).double().cpu().numpy()
    ax = [g["o"][a] + g["h"][a] * stride * np.arange(m[a]) for a in range(3)]

    def emb(a, b, c):
        if coord == 0:
            return np.stack(np.broadcast_arrays(a, b, c), -1)
        return np.stack([a * np.cos(b) * np.cos(c), a * np.cos(b) * np.sin(c), a * np.sin(b) + 0.0 * c], -1)

    X = emb(ax[0][:, None, None], ax[1][None, :, None], ax[2][None, None, :])
    cut = tuple(slice(None, None, stride) for _ in range(3))
    for q in range(2):
        d = np.linalg.norm(X - emb(*src[q]), axis=-1)
        ref = np.stack([(s[cut] / par[q, 0] - 1) * 5, xi[cut] * 25, eta[cut] * 25, d * 0.01], -1)
        got = f[q, :m[0], :m[1], :m[2], :4]
        assert np.all(np.abs(got - ref) <= 2.0 ** -8 * np.abs(ref) + 1e-7)
    rest = f.copy()
    rest[:, :m[0], :m[1], :m[2], :4] = 0.0
    assert np.all(rest == 0.0)
    pred = rng.standard_normal((2,) + dims).astype(np.float32)
    pred[1, 0, 0, 0] = np.nan
    tau = nn.warm_init(g, torch.as_tensor(pred).cuda(), stride).cpu().numpy().reshape((2,) + n)
    ref = pred[:, :m[0], :m[1], :m[2]].astype(np.float64)
    for a in range(3):
        i = np.arange(n[a])
        b = np.minimum(i // stride, m[a] - 1)
        c = np.minimum(b + 1, m[a] - 1)
        w = np.where(c == b, 0.0, (i - b * stride) / stride).reshape([-1 if e == a + 1 else 1 for e in range(4)])
        lo_, hi_ = np.take(ref, b, a + 1), np.take(ref, c, a + 1)
        ref = np.where(w == 0.0, lo_, (1 - w) * lo_ + w * hi_)
    ref = np.where(np.isnan(ref), 1.0, np.clip(1 + ref / 10, 0.25, 4.0))
    assert np.allclose(tau, ref, rtol=1e-12, atol=1e-12)
