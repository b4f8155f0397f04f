"""Tile variants of the convolution kernels, at the sizes where each takes
over and where tiles are ragged.  Bounds as in test_gpu_unet: FP32
accumulation within 1e-5 of the sum of absolute products, bf16 outputs within
one bf16 ulp (2^-8 relative) on top."""
import numpy as np
import pytest

from oracle import unet_ref as R
from test_gpu_unet import U, bf, dev, host  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,h,w,cin,cout", [
    (16, 261, 16, 32, 64),    # 64 x 64 wave tiles, 16 columns, last tile row partial
    (1, 130, 129, 64, 128),   # 32 x 64 wave tiles, last tile row and column partial
    (3, 37, 53, 64, 192),     # 32 x 32 wave tiles, all weights of a tap row per stage
    (1, 5, 33, 384, 64),      # the same with the shorter weight stages (LDS)
    (2, 9, 7, 96, 32),        # 32 output channels, image smaller than a tile
    (1, 259, 257, 96, 32),    # 32 output channels, 64-pixel wave tiles
    (1, 3, 5, 1216, 64),      # more input channels than LDS holds
    (1, 1, 1, 1216, 32),      # one pixel
])
def test_conv_tiles(U, n, h, w, cin, cout):
    import torch
    print("[gpu-case] conv tiles", n, h, w, cin, cout, flush=True)
    rng = np.random.default_rng(20)
    x, wt = bf(rng, n, h, w, cin), bf(rng, cout, 9, cin, scale=0.1)
    b = rng.standard_normal(cout).astype(np.float32).astype(np.float64)
    ref, bound = R.conv3x3(x, wt, b), R.conv3x3(np.abs(x), np.abs(wt)) + np.abs(b)
    xd, wd, bd = dev(x, torch.bfloat16), dev(wt, torch.bfloat16), dev(b, torch.float32)
    # output rows wider than the layer: the neighbours' channels stay as they are
    y = torch.full((n, h, w, cout + 8), 7.0, device="cuda", dtype=torch.float32)
    U.conv3x3_fwd(xd, wd, bd, cout, out_f32=True, y=y)
    assert (np.abs(host(y)[..., :cout] - ref) <= 1e-5 * bound + 1e-6).all()
    assert (host(y)[..., cout:] == 7.0).all()
    yr = torch.full((n, h, w, cout + 8), 7.0, device="cuda", dtype=torch.bfloat16)
    U.conv3x3_fwd(xd, wd, bd, cout, relu=True, y=yr)
    refr = np.maximum(ref, 0)
    assert (np.abs(host(yr)[..., :cout] - refr) <= 2 ** -8 * refr + 1e-5 * bound + 1e-6).all()
    assert (host(yr)[..., cout:] == 7.0).all()


@pytest.mark.parametrize("n,h,w,cin,cout", [(33, 64, 64, 64, 64), (9, 64, 128, 96, 32),
                                            (40, 16, 16, 128, 128)])
def test_conv_variants_agree_bit_for_bit(U, n, h, w, cin, cout):
    """One image alone takes another wave tile than the batch it is part of;
    the sums run in the same order."""
    import torch
    print("[gpu-case] conv variants", n, h, w, cin, cout, flush=True)
    rng = np.random.default_rng(21)
    x, wt = dev(bf(rng, n, h, w, cin), torch.bfloat16), dev(bf(rng, cout, 9, cin), torch.bfloat16)
    y = U.conv3x3_fwd(x, wt, None, cout, out_f32=True)
    for k in (0, n - 1):
        one = U.conv3x3_fwd(x[k:k + 1].contiguous(), wt, None, cout, out_f32=True)
        assert torch.equal(one[0], y[k])


@pytest.mark.parametrize("n,h,w,cin,cout", [
    (1, 1, 1, 32, 32),        # one pixel
    (2, 13, 35, 32, 96),      # 32-column tiles, ragged both ways, one share per tile
    (3, 21, 11, 64, 64),      # 16-column tiles
    (24, 64, 64, 64, 64),     # many pixel tiles: 64 x 64 channel tiles or shared partial sums
    (64, 40, 12, 128, 64),    # the same with 16-column tiles
    (5, 33, 65, 96, 128),     # 96 input channels
])
def test_weight_gradient_tiles(U, n, h, w, cin, cout):
    import torch
    print("[gpu-case] weight gradient tiles", n, h, w, cin, cout, flush=True)
    rng = np.random.default_rng(22)
    dyf, xf = bf(rng, n, h, w, cout + 8), bf(rng, n, h, w, cin + 32)
    dy, x = dyf[..., :cout], xf[..., :cin]
    dw_ref, db_ref = R.conv3x3_bwd_weight(dy, x)
    bound, _ = R.conv3x3_bwd_weight(np.abs(dy), np.abs(x))
    dw, db = U.conv3x3_bwd_weight(dev(dyf, torch.bfloat16), dev(xf, torch.bfloat16), cin, cout)
    assert (np.abs(host(dw) - dw_ref) <= 1e-5 * bound + 1e-6).all()
    assert (np.abs(host(db) - db_ref) <= 1e-5 * np.abs(dy).reshape(-1, cout).sum(0) + 1e-6).all()


def test_images_of_two_gigabytes(U):
    """A pixel stride so large that an image spans 2 GB: loads with 64-bit
    addresses, the same sums."""
    import torch
    print("[gpu-case] 2 GB images", flush=True)
    rng = np.random.default_rng(23)
    x, dy = bf(rng, 1, 1, 3, 32), bf(rng, 1, 1, 3, 64)
    wt = bf(rng, 64, 9, 32, scale=0.1)
    xd = torch.zeros((1, 1, 3, 2 ** 29), device="cuda", dtype=torch.bfloat16)
    xd[..., :32] = dev(x, torch.bfloat16)
    y = U.conv3x3_fwd(xd, dev(wt, torch.bfloat16), None, 64, out_f32=True)
    bound = R.conv3x3(np.abs(x), np.abs(wt))
    assert (np.abs(host(y) - R.conv3x3(x, wt)) <= 1e-5 * bound + 1e-6).all()
    dw, _ = U.conv3x3_bwd_weight(dev(dy, torch.bfloat16), xd, 32, 64)
    dw_ref, _ = R.conv3x3_bwd_weight(dy, x)
    bound, _ = R.conv3x3_bwd_weight(np.abs(dy), np.abs(x))
    assert (np.abs(host(dw) - dw_ref) <= 1e-5 * bound + 1e-6).all()


def layered_forward(U, params, x0):
    """The network from the single-layer functions (weights as rows)."""
    import torch
    lay, _ = R.param_layout()

    def conv(k, x, relu=True):
        w_off, b_off, ci, co = lay[k]
        w = params[w_off:w_off + 9 * ci * co].to(torch.bfloat16).reshape(co, 9, ci).contiguous()
        return U.conv3x3_fwd(x.contiguous(), w, params[b_off:b_off + co].contiguous(), co,
                             relu=relu, out_f32=not relu)

    def up_cat(a, skip):
        return torch.cat([U.up2_fwd(a), skip], dim=3)

    e0 = conv(1, conv(0, x0))
    e1 = conv(3, conv(2, U.pool2_fwd(e0)))
    e2 = conv(5, conv(4, U.pool2_fwd(e1)))
    b3 = conv(7, conv(6, U.pool2_fwd(e2)))
    d2 = conv(9, conv(8, up_cat(b3, e2)))
    d1 = conv(11, conv(10, up_cat(d2, e1)))
    return conv(14, conv(13, conv(12, up_cat(d1, e0))), relu=False)


@pytest.mark.parametrize("res,n", [(8, 1), (24, 3), (128, 1), (128, 3), (128, 16)])
def test_network_equals_its_layers(U, res, n):
    """The network's forms of a convolution (weights in fragment order, fused
    pooling and upsampling, one or two tiles per wavefront by batch) give the
    bits of the single layers, also after the weights have changed."""
    import torch
    print("[gpu-case] network layers", res, n, flush=True)
    rng = np.random.default_rng(res + n)
    net = U.UNet(max_batch=n, res=res, seed=5)
    x0 = dev(bf(rng, n, res, res, 32), torch.bfloat16)
    target = dev(rng.standard_normal((n, res, res, 3)), torch.float32)
    fluid = torch.ones((n, res, res), dtype=torch.uint8, device="cuda")
    for _ in range(2):
        want = layered_forward(U, dev(net.params(), torch.float32), x0)
        assert torch.equal(net.forward(x0), want)
        net.train_step(x0, target, fluid, 1e-3)
    net.close()


@pytest.mark.parametrize("side", [3, 8, 127, 128, 129, 200])
def test_mass_fix_and_maps_sizes(U, side):
    """Cases below, at and above what the threads of a case keep in registers
    (16384 nodes), ragged ones among them; bounds as in test_gpu_unet."""
    import torch
    rng = np.random.default_rng(side)
    solid = (rng.random((3, side, side)) > 0.8).astype(np.uint8)
    solid[2] = 1                      # a case without fluid nodes
    cp = np.array([[100.0, 0.3, 0.05], [450.0, 1.0, 0.1], [50.0, 0.5, 0.1]], np.float32)
    for res in (8, 40):
        x0 = host(U.make_input(dev(solid, torch.uint8), dev(cp, torch.float32), res))
        np.testing.assert_allclose(x0, R.bf16(R.make_input(solid, cp.astype(np.float64), res)),
                                   rtol=2 ** -8, atol=0)
    for ld in (3, 8, 32):             # pixels read as single floats and as four
        out = rng.standard_normal((3, 16, 16, ld)).astype(np.float32).astype(np.float64)
        got = U.fields_from_output(dev(out, torch.float32), dev(cp, torch.float32),
                                   dev(solid, torch.uint8))
        ref = R.fields_from_output(out, cp.astype(np.float64), solid)
        for g, r, tol in zip(got, ref, (2e-6, 1e-6, 1e-6)):
            np.testing.assert_allclose(host(g), r, rtol=0, atol=tol)


def layered_gradients(U, params, x0, target, fluid):
    """Weight gradients of all layers from the single-layer functions."""
    import torch
    lay, _ = R.param_layout()
    ws = [params[w:w + 9 * ci * co].to(torch.bfloat16).reshape(co, 9, ci).contiguous()
          for w, _, ci, co in lay]
    bs = [params[b:b + co].contiguous() for _, b, _, co in lay]
    xs, grads = {}, {}

    def conv(k, x, relu=True):
        xs[k] = x.contiguous()
        return U.conv3x3_fwd(xs[k], ws[k], bs[k], lay[k][3], relu=relu, out_f32=not relu)

    def back(k, dy, dx=True):
        ci, co = lay[k][2:]
        grads[k] = U.conv3x3_bwd_weight(dy, xs[k], ci, co)[0]
        return U.conv3x3_bwd_data(dy, ws[k], ci) if dx else None

    a0 = conv(0, x0)
    e0 = conv(1, a0)
    a1 = conv(2, U.pool2_fwd(e0))
    e1 = conv(3, a1)
    a2 = conv(4, U.pool2_fwd(e1))
    e2 = conv(5, a2)
    a3 = conv(6, U.pool2_fwd(e2))
    b3 = conv(7, a3)
    c2 = conv(8, torch.cat([U.up2_fwd(b3), e2], 3))
    d2 = conv(9, c2)
    c1 = conv(10, torch.cat([U.up2_fwd(d2), e1], 3))
    d1 = conv(11, c1)
    c0 = conv(12, torch.cat([U.up2_fwd(d1), e0], 3))
    d0 = conv(13, c0)
    _, dout = U.mse_loss(conv(14, d0, relu=False), target, fluid)
    relu = lambda d, y: U.relu_bwd(d.contiguous(), y)   # noqa: E731
    g = back(12, relu(back(13, relu(back(14, dout), d0)), c0))
    s0, g = g[..., 64:], relu(U.up2_bwd(g[..., :64].contiguous()), d1)
    g = back(10, relu(back(11, g), c1))
    s1, g = g[..., 128:], relu(U.up2_bwd(g[..., :128].contiguous()), d2)
    g = back(8, relu(back(9, g), c2))
    s2, g = g[..., 256:], relu(U.up2_bwd(g[..., :256].contiguous()), b3)
    g = back(6, relu(back(7, g), a3))
    g = relu(U.pool2_bwd(g, s2.contiguous()), e2)
    g = back(4, relu(back(5, g), a2))
    g = relu(U.pool2_bwd(g, s1.contiguous()), e1)
    g = back(2, relu(back(3, g), a1))
    g = relu(U.pool2_bwd(g, s0.contiguous()), e0)
    back(0, relu(back(1, g), a0), dx=False)
    return grads


@pytest.mark.parametrize("res,n", [(16, 2), (128, 3), (3360, 1)])
def test_network_gradients_equal_its_layers(U, res, n):
    """The backward pass (fused masks, grouped weight gradients, fragment
    weights) against the single layers; 3360^2 has images of more than 2 GB in
    the finest level, where every fused form takes the general kernel.  The
    input gradients are the same bits, the weight gradients sum the same
    products in FP32 over another split: 20 eps of the sum of absolute products
    (chains of about 400 additions), taken as at most 800 largest entries."""
    import torch
    print("[gpu-case] network gradients", res, n, flush=True)
    rng = np.random.default_rng(res)
    net = U.UNet(max_batch=n, res=res, seed=6)
    small = rng.standard_normal((n, 16, 16, 32))
    rep = (res + 15) // 16
    x0 = dev(R.bf16(np.tile(small, (1, rep, rep, 1))[:, :res, :res]), torch.bfloat16)
    target = dev(np.tile(small[..., :3], (1, rep, rep, 1))[:, :res, :res], torch.float32)
    fluid = torch.ones((n, res, res), dtype=torch.uint8, device="cuda")
    params = dev(net.params(), torch.float32)
    net.backward(x0, target, fluid)
    got = net.grads()
    want = layered_gradients(U, params, x0, target, fluid)
    net.close()
    lay, _ = R.param_layout()
    for k, (w, _, ci, co) in enumerate(lay):
        ref = want[k].float().cpu().numpy().reshape(-1)
        err = np.abs(got[w:w + 9 * ci * co] - ref).max()
        assert err <= 1e-3 * np.abs(ref).max(), (k, err, np.abs(ref).max())


@pytest.mark.parametrize("n,h,w,cin,cout", [
    (3, 9, 37, 416, 32),      # a tile of 16 columns, where 32 do not fit
    (2, 17, 33, 640, 64),
    (1, 257, 259, 704, 64),   # no tile fits: 64-pixel wave tiles, last block partial
    (1, 263, 250, 1024, 32),  # the same with 32 output channels
])
def test_wide_convolutions_equal_narrow_ones(U, n, h, w, cin, cout):
    """Many input channels.  The outer ones are zero, so the result is that of the
    inner 64 alone, which another kernel takes: the same bits, as zeros add
    nothing to the sums."""
    import torch
    print("[gpu-case] wide", n, h, w, cin, cout, flush=True)
    rng = np.random.default_rng(24)
    x = torch.zeros((n, h, w, cin), device="cuda", dtype=torch.bfloat16)
    wt = torch.zeros((cout, 9, cin), device="cuda", dtype=torch.bfloat16)
    xs, ws = dev(bf(rng, n, h, w, 64), torch.bfloat16), dev(bf(rng, cout, 9, 64), torch.bfloat16)
    x[..., :64], wt[..., :64] = xs, ws
    b = dev(rng.standard_normal(cout), torch.float32)
    for kw in (dict(out_f32=True), dict(relu=True)):
        assert torch.equal(U.conv3x3_fwd(x, wt, b, cout, **kw), U.conv3x3_fwd(xs, ws, b, cout, **kw))
    # and against the reference at a corner with every channel
    xr, wr = bf(rng, 1, 5, 6, cin), bf(rng, cout, 9, cin, scale=0.1)
    x[:1, :5, :6] = dev(xr, torch.bfloat16)
    got = host(U.conv3x3_fwd(x, dev(wr, torch.bfloat16), None, cout, out_f32=True))[0, :4, :5]
    bound = R.conv3x3(np.abs(xr), np.abs(wr))[0, :4, :5]
    assert (np.abs(got - R.conv3x3(xr, wr)[0, :4, :5]) <= 1e-5 * bound + 1e-6).all()


@pytest.mark.parametrize("n,h,w,cin,cout", [
    (2000, 1, 1, 32, 64), (1400, 3, 2, 96, 32), (4100, 4, 4, 64, 128), (16400, 1, 4, 32, 32),
    (3300, 9, 9, 64, 128),
])
def test_many_small_images_equal_single_ones(U, n, h, w, cin, cout):
    """Kernels without tiles (small and large form), and a smaller tile: the bits
    of one image alone."""
    import torch
    print("[gpu-case] small images", n, h, w, cin, cout, flush=True)
    rng = np.random.default_rng(25)
    x, wt = dev(bf(rng, n, h, w, cin), torch.bfloat16), dev(bf(rng, cout, 9, cin), torch.bfloat16)
    for kw in (dict(out_f32=True), dict(relu=True)):
        y = U.conv3x3_fwd(x, wt, None, cout, **kw)
        for k in (0, n // 2, n - 1):
            one = U.conv3x3_fwd(x[k:k + 1].contiguous(), wt, None, cout, **kw)
            assert torch.equal(one[0], y[k])


@pytest.mark.parametrize("res,n", [(8, 1100), (16, 1030)])
def test_network_of_many_small_samples(U, res, n):
    """Levels of 1 x 1 to 16 x 16: the fused forms (pooling, upsampling, masks) in
    the kernels without tiles give the bits of the single layers, and a sample the
    bits it has alone."""
    import torch
    print("[gpu-case] network, small samples", res, n, flush=True)
    rng = np.random.default_rng(res)
    net = U.UNet(max_batch=n, res=res, seed=7)
    x0 = dev(bf(rng, n, res, res, 32), torch.bfloat16)
    want = layered_forward(U, dev(net.params(), torch.float32), x0)
    got = net.forward(x0)
    assert torch.equal(got, want)
    for k in (0, n - 1):
        assert torch.equal(net.forward(x0[k:k + 1].contiguous())[0], want[k])
    net.close()


@pytest.mark.parametrize("n,h,w,cin,cout", [(2, 13, 35, 32, 64), (1, 16, 16, 32, 32),
                                            (3, 21, 11, 64, 32), (1, 33, 48, 32, 32)])
def test_weight_gradient_of_inputs_that_are_not_finite(U, n, h, w, cin, cout):
    """An infinity in the last row or column reaches the taps that see it and no
    others: the padding of the pixel tiles adds nothing."""
    import torch
    import torch.nn.functional as F
    print("[gpu-case] weight gradient, infinities", n, h, w, cin, cout, flush=True)
    rng = np.random.default_rng(26)
    x, dy = bf(rng, n, h, w, cin), np.abs(bf(rng, n, h, w, cout)) + 0.5
    x[0, h - 1, w // 2, 1] = np.inf
    x[n - 1, h // 2, w - 1, 2] = -np.inf
    x[0, h - 1, w - 1, 3] = np.inf
    dw, db = U.conv3x3_bwd_weight(dev(dy, torch.bfloat16), dev(x, torch.bfloat16), cin, cout)
    # the sums themselves, tap by tap, over the pixels a tap sees
    dyr = host(dev(dy, torch.bfloat16))
    want = np.zeros((cout, 9, cin))
    xp = np.zeros((n, h + 2, w + 2, cin))
    xp[:, 1:-1, 1:-1] = x
    for t in range(9):
        view = xp[:, t // 3:t // 3 + h, t % 3:t % 3 + w]
        inside = np.zeros((n, h + 2, w + 2, 1), bool)
        inside[:, 1:-1, 1:-1] = True
        inside = inside[:, t // 3:t // 3 + h, t % 3:t % 3 + w, 0]
        want[:, t] = dyr[inside].T @ view[inside]
    got = host(dw)
    finite = np.isfinite(want)
    assert 0 < (~finite).sum() < finite.size
    np.testing.assert_array_equal(np.isfinite(got), finite)
    np.testing.assert_array_equal(got[~finite], want[~finite])
    bound = np.abs(dyr).reshape(-1, cout).sum(0).max() * np.abs(x[np.isfinite(x)]).max()
    assert np.abs(got[finite] - want[finite]).max() <= 1e-5 * bound
    assert np.isfinite(host(db)).all()


@pytest.mark.parametrize("n,h,w", [
    (1, 1, 1), (63, 1, 1), (65, 1, 1), (300, 1, 1), (26, 2, 2), (40, 3, 5), (10, 4, 4), (9, 4, 4),
    (5, 7, 7), (4, 7, 7), (7, 6, 1), (9, 1, 7), (3, 5, 40), (5, 40, 6), (17, 1, 33), (3, 200, 1),
    (3, 7, 8), (3, 8, 7),
])
def test_weight_gradient_of_small_images(U, n, h, w):
    """Several images to a pixel tile, full and partly filled, packed along one side
    or both; image sizes around the largest that is packed."""
    import torch
    print("[gpu-case] weight gradient, small images", n, h, w, flush=True)
    rng = np.random.default_rng(27)
    cin, cout = 64, 32
    dyf, xf = bf(rng, n, h, w, cout + 8), bf(rng, n, h, w, cin + 32)
    dy, x = dyf[..., :cout], xf[..., :cin]
    dw_ref, db_ref = R.conv3x3_bwd_weight(dy, x)
    bound, _ = R.conv3x3_bwd_weight(np.abs(dy), np.abs(x))
    dw, db = U.conv3x3_bwd_weight(dev(dyf, torch.bfloat16), dev(xf, torch.bfloat16), cin, cout)
    assert (np.abs(host(dw) - dw_ref) <= 1e-5 * bound + 1e-6).all()
    assert (np.abs(host(db) - db_ref) <= 1e-5 * np.abs(dy).reshape(-1, cout).sum(0) + 1e-6).all()
    # an infinity stays in its image
    x[n // 2, h - 1, w - 1, 0] = np.inf
    xf[..., :cin] = x
    dwi, _ = U.conv3x3_bwd_weight(dev(dyf, torch.bfloat16), dev(xf, torch.bfloat16), cin, cout)
    got = host(dwi)
    np.testing.assert_array_equal(got[:, :, 1:], host(dw)[:, :, 1:])
    sees = [t for t in range(9) if 0 <= h - 1 - (t // 3 - 1) < h and 0 <= w - 1 - (t % 3 - 1) < w]
    assert not np.isfinite(got[:, sees, 0]).any()
    assert np.isfinite(got[:, [t for t in range(9) if t not in sees], 0]).all()


def test_small_images_with_a_wide_stride(U):
    """Images of a few pixels whose pixel stride makes a tile of them 2 GB."""
    import torch
    print("[gpu-case] small images, 2 GB tile", flush=True)
    rng = np.random.default_rng(28)
    n, ld = 9, 2 ** 27 + 8
    x, dy = bf(rng, n, 1, 1, 32), bf(rng, n, 1, 1, 32)
    xd = torch.empty(n * ld, device="cuda", dtype=torch.bfloat16).view(n, 1, 1, ld)
    xd[..., :32] = dev(x, torch.bfloat16)
    dw, _ = U.conv3x3_bwd_weight(dev(dy, torch.bfloat16), xd, 32, 32)
    dw_ref, _ = R.conv3x3_bwd_weight(dy, x)
    bound, _ = R.conv3x3_bwd_weight(np.abs(dy), np.abs(x))
    assert (np.abs(host(dw) - dw_ref) <= 1e-5 * bound + 1e-6).all()
