"""Weight and bias gradients of the whole network (one grouped launch, one launch
of split sums) against its single layers, entry by entry."""
import numpy as np
import pytest

from oracle import unet_ref as R
from test_gpu_unet import U, bf, dev  # noqa: F401
from test_gpu_unet_tiles import layered_gradients

pytestmark = pytest.mark.gpu


class Recorder:
    """The functions of the library; the weight gradients' results are kept, with
    the sums of absolute products that bound their rounding."""

    def __init__(self, lib):
        self.lib, self.calls = lib, []

    def __getattr__(self, name):
        return getattr(self.lib, name)

    def conv3x3_bwd_weight(self, dy, x, cin, cout):
        got = self.lib.conv3x3_bwd_weight(dy, x, cin, cout)
        self.calls.append((got, self.lib.conv3x3_bwd_weight(dy.abs(), x.abs(), cin, cout)))
        return got


@pytest.mark.parametrize("res,n", [
    (8, 1), (8, 70), (16, 2), (40, 5),   # several images to a tile in the coarse levels
    (128, 1),                            # few splits in every layer
    (128, 3), (128, 16),                 # more than 16 splits in the fine levels
])
def test_gradients_of_every_layer(U, res, n):
    """Both sides sum the same products in FP32 in another order.  A chain holds at
    most 512 additions (12 tiles of 2 rows of 16 pixels, 8 wavefronts, the
    splits), so each side is within 512 x 2^-24 of the sum of absolute products."""
    import torch
    print("[gpu-case] network gradients, every layer", res, n, flush=True)
    rng = np.random.default_rng(1000 * res + n)
    net = U.UNet(max_batch=n, res=res, seed=8)
    x0 = dev(bf(rng, n, res, res, 32), torch.bfloat16)
    target = dev(rng.standard_normal((n, res, res, 3)), torch.float32)
    fluid = dev((rng.random((n, res, res)) > 0.2).astype(np.uint8), torch.uint8)
    params = dev(net.params(), torch.float32)
    net.backward(x0, target, fluid)
    got = net.grads()
    net.close()
    rec = Recorder(U)
    layered_gradients(rec, params, x0, target, fluid)
    lay, _ = R.param_layout()
    assert len(rec.calls) == len(lay)
    for k, ((dw, db), (bw, bb)) in zip(reversed(range(len(lay))), rec.calls):
        w, b, ci, co = lay[k]
        for lo, ref, bound in ((w, dw, bw), (b, db, bb)):
            ref = ref.double().cpu().numpy().reshape(-1)
            err = np.abs(got[lo:lo + ref.size] - ref)
            limit = 2 * 512 * 2.0 ** -24 * bound.double().cpu().numpy().reshape(-1)
            assert (err <= limit + 1e-30).all(), (k, lo == b, (err - limit).max())
        assert np.abs(got[b:b + co]).max() > 0
