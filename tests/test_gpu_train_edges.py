"""Gradients at the sizes where the weight-gradient kernels can go wrong:
channel counts that leave a 16- or 32-channel block partly empty, images that
are no multiple of the 8 x 16 tiles, several pixel tiles per workgroup, runs
of pixels that end inside a wavefront's share; against the fp64 oracle, per
tensor, at the bound of the other gradient tests.  The networks' weights are
positive and small, so that no pre-activation lies near zero (a ReLU mask
that differs from fp64's would say nothing about the sums)."""
import numpy as np
import pytest

from synth.weights import adapter_params, he_normal_params
from tests.helpers import log, to_dev, to_host
from tests.test_gpu_train import GRAD_REL, _batch, _split
from tests.test_gpu_train_adapters import _adapter_tensors

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2604_03748_amd import lnm

    return lnm.Context(0)


def _params(levels, base):
    return np.abs(he_normal_params(levels, base, seed=5, bias="uniform")) * np.float32(0.05)


def _check(got, ref, what):
    for k in ref:
        n = np.linalg.norm(ref[k])
        rel = np.linalg.norm(got[k] - ref[k]) / max(n, 1e-30)
        assert rel <= GRAD_REL or n == 0.0 == np.linalg.norm(got[k]), (what, k, rel)


@pytest.mark.parametrize("levels,base,B,H,W", [(2, 48, 1, 10, 34), (2, 80, 1, 6, 18), (2, 16, 3, 18, 50),
                                               (2, 16, 1, 320, 320), (2, 16, 3, 232, 238)])
def test_trunk_gradient(ctx, orc, levels, base, B, H, W):
    from paper_2604_03748_amd import lnm

    params = _params(levels, base)
    g, t = _batch(B, H, W, base + W)
    tr = lnm.Trainer(ctx, levels, base, params)
    loss, grad = tr.grad(to_dev(g), to_dev(t))
    ref_loss, ref = orc.unet_loss_grad(params, levels, base, g.astype(np.float64), t.astype(np.float64))
    log(f"L{levels}b{base} {B}x{H}x{W}: loss {float(to_host(loss)[0]):.8g} vs {ref_loss:.8g}")
    assert abs(float(to_host(loss)[0]) - ref_loss) <= 1e-5 * ref_loss
    _check(_split(to_host(grad), levels, base), _split(ref, levels, base), (base, H, W))


@pytest.mark.parametrize("base,B,H,W", [(16, 3, 18, 50), (48, 1, 10, 34), (64, 1, 20, 38)])
def test_adapter_gradient(ctx, orc, base, B, H, W):
    from paper_2604_03748_amd import lnm

    params = _params(2, base)
    ad = adapter_params(base, seed=6)
    g, t = _batch(B, H, W, base + W)
    tr = lnm.Trainer(ctx, 2, base, params)
    tr.attach_adapters(ad)
    tr.grad(to_dev(g), to_dev(t))
    got = to_host(tr.adapter_grad())
    ref = orc.adapters_loss_grad(params, 2, base, ad, g.astype(np.float64), t.astype(np.float64))[2]
    _check(_adapter_tensors(got, base), _adapter_tensors(ref, base), (base, H, W))


def test_activations_past_bf16(ctx, orc):
    """First-layer outputs from 3e38 to 3.4e38, which the three-piece splits'
    plain form cannot hold (it rounds the largest to infinity): the second
    layer's weight gradient, which sums products of them."""
    from paper_2604_03748_amd import lnm

    base, params = 16, _params(2, 16)
    parts = _split(params, 2, base)
    parts["enc0a.w"][:] = 0.0
    parts["enc0a.w"].reshape(base, 3, 9)[np.arange(base), np.arange(base) % 3, 4] = 3.4e38
    parts["enc0a.b"][:] = 0.0
    parts["enc0b.w"][:] = (1.0 + parts["enc0b.w"]) * 1e-36  # outputs near 2e4
    parts["bot1a.w"][:] *= 1e-4
    parts["dec0a.w"].reshape(base, 3 * base, 9)[:, :base] *= 1e-4
    g, t = _batch(1, 24, 40, 7)
    g[:] = np.random.default_rng(8).choice([0.0, 0.9, 1.0], g.shape)
    tr = lnm.Trainer(ctx, 2, base, params)
    _, grad = tr.grad(to_dev(g), to_dev(t))
    ref = orc.unet_loss_grad(params, 2, base, g.astype(np.float64), t.astype(np.float64))[1]
    got, ref = (_split(v.astype(np.float64), 2, base)["enc0b.w"] for v in (to_host(grad), ref))
    assert np.isfinite(got).all() and np.abs(ref).max() > 1e20
    assert np.linalg.norm(got - ref) <= GRAD_REL * np.linalg.norm(ref)
