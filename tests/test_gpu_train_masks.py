"""Gradients through ReLU masks that vary from pixel to pixel and from channel
to channel, at sizes with partial tiles and partly empty channel blocks,
against the fp64 oracle.  Each guide channel is 0 or 3 at random; the layers'
centre taps join channels of one of three classes, the biases lie between the
sums that arise, and the other taps are small: every pre-activation is at
least MARGIN away from zero (checked here in fp64), so the masks are the same
in fp32, and one read from another pixel or channel changes the gradient by
far more than the bound."""
import numpy as np
import pytest

from synth.weights import n_params, unet_layers
from tests.helpers import log, to_dev, to_host
from tests.test_gpu_train import _batch, _split
from tests.test_gpu_train_edges import _check

pytestmark = pytest.mark.gpu

MARGIN = 0.02

@pytest.fixture(scope="module")
def ctx():
    from paper_2604_03748_amd import lnm

    return lnm.Context(0)


def _params(levels, base):
    """Output channel o takes the input channels of its class (c % 3 == o % 3)."""
    rng = np.random.default_rng(base)
    out = np.empty(n_params(levels, base), dtype=np.float32)
    at = 0
    for name, ci, co, k in unet_layers(levels, base):
        w = rng.uniform(-1.0, 1.0, (co, ci, k * k)) * 0.02 / (k * k * ci)
        if k == 3:
            same = np.arange(ci) % 3 == np.arange(co)[:, None] % 3
            scale = 1.0 if ci == 3 else 1.6 / same.sum(1, keepdims=True)
            w[:, :, 4] += np.where(same, scale * rng.uniform(0.9, 1.1, (co, ci)), 0.0)
        else:
            w = rng.uniform(-1.0, 1.0, w.shape) / ci
        out[at:at + w.size] = w.ravel()
        out[at + w.size:at + w.size + co] = -0.3 * rng.uniform(0.9, 1.1, co) if k == 3 else 0.1
        at += w.size + co
    return out


def _preactivations(params, levels, base, g):
    import torch

    t, off = torch.from_numpy(params).double(), 0
    pre, it = [], iter(unet_layers(levels, base))

    def conv(x):
        nonlocal off
        _, ci, co, k = next(it)
        n = co * ci * k * k
        z = torch.nn.functional.conv2d(x, t[off:off + n].reshape(co, ci, k, k), t[off + n:off + n + co], padding=1)
        off += n + co
        pre.append(z)
        return z.clamp(min=0)

    x, skips = torch.from_numpy(g).double().permute(0, 3, 1, 2), []
    for l in range(levels):
        x = conv(conv(torch.nn.functional.max_pool2d(x, 2) if l else x))
        skips.append(x)
    for l in range(levels - 2, -1, -1):
        x = conv(conv(torch.cat([skips[l], x.repeat_interleave(2, 2).repeat_interleave(2, 3)], 1)))
    return pre


@pytest.mark.parametrize("levels,base,B,H,W", [(2, 48, 1, 10, 34), (2, 80, 1, 6, 18), (3, 16, 2, 20, 36),
                                               (2, 32, 3, 66, 70), (2, 16, 24, 130, 34)])
def test_gradient_through_mixed_masks(ctx, orc, levels, base, B, H, W):
    from paper_2604_03748_amd import lnm

    params = _params(levels, base)
    g, t = _batch(B, H, W, base + W)
    g[:] = 3.0 * (np.random.default_rng(base + H).random(g.shape) < 0.12)
    for z in _preactivations(params, levels, base, g):
        assert float(z.abs().min()) >= MARGIN
        assert 0.05 <= float((z > 0).double().mean()) <= 0.95
    tr = lnm.Trainer(ctx, levels, base, params)
    loss, grad = tr.grad(to_dev(g), to_dev(t))
    ref_loss, ref = orc.unet_loss_grad(params, levels, base, g.astype(np.float64), t.astype(np.float64))
    log(f"masks L{levels}b{base} {B}x{H}x{W}: loss {float(to_host(loss)[0]):.8g} vs {ref_loss:.8g}")
    assert abs(float(to_host(loss)[0]) - ref_loss) <= 1e-5 * ref_loss
    _check(_split(to_host(grad), levels, base), _split(ref, levels, base), (base, H, W))
