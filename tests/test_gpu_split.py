"""The fp32 convolutions on the bf16 matrix cores (three-piece splits): each
tile height and channel count that leaves a block partly empty against the
fp64 oracle, and values that bf16 cannot hold (infinities, finite values past
bf16's largest) against the same layers in fp64 torch."""
import numpy as np
import pytest

from synth.weights import he_normal_params, unet_layers
from tests.helpers import check_net, log, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2604_03748_amd import lnm

    return lnm.Context(0)


# (8 x 256^2 and the 64 small images take 16-row tiles, 24 x 48^2 8-row tiles, the others 4-row ones)
@pytest.mark.parametrize("levels,base,B,H,W", [(2, 16, 1, 6, 10), (3, 48, 1, 20, 36), (2, 16, 24, 48, 48),
                                               (2, 32, 64, 34, 18), (2, 16, 8, 256, 256)])
def test_tiles(ctx, orc, levels, base, B, H, W):
    import torch
    from paper_2604_03748_amd import lnm

    params = he_normal_params(levels, base, seed=4, bias="uniform")
    g = (np.random.default_rng(B + W).random((B, H, W, 3)) * np.array([2.5, 1.0, 3.5])).astype(np.float32)
    net = lnm.Net(ctx, levels, base, params)
    logits = torch.empty((B, H, W, 6), device="cuda")
    lm = net.infer(to_dev(g), logits=logits)
    fused = net.infer(to_dev(g))
    pick = sorted({0, B - 1})
    ref, ref_z = orc.unet_forward(params, levels, base, g[pick].astype(np.float64))
    check_net(to_host(lm)[pick], ref.reshape(len(pick), H, W, 6), to_host(logits)[pick],
              ref_z.reshape(len(pick), H, W, 6), f"split L{levels}b{base} {B}x{H}x{W}")
    assert np.abs(to_host(fused) - to_host(lm)).max() <= 1e-6  # the head in the last layer's epilogue


def _torch_logits(params, levels, base, g):
    """The network in fp64 with ReLU(NaN) = 0, as max(x, 0) of the kernels gives."""
    import torch

    layers, at, prm = unet_layers(levels, base), 0, []
    for _, ci, co, k in layers:
        n = co * ci * k * k
        prm.append((torch.tensor(params[at:at + n].astype(np.float64)).reshape(co, ci, k, k),
                    torch.tensor(params[at + n:at + n + co].astype(np.float64))))
        at += n + co
    it = iter(prm)

    def conv(x):
        w, b = next(it)
        cols = torch.nn.functional.unfold(x, 3, padding=1)  # [B][ci * 9][HW]
        y = (w.reshape(1, w.shape[0], -1) @ cols).reshape(x.shape[0], w.shape[0], *x.shape[2:]) + b[:, None, None]
        return torch.where(y > 0, y, torch.zeros_like(y))

    x, skips = torch.tensor(g.astype(np.float64)).permute(0, 3, 1, 2), []
    for l in range(levels):
        if l:
            x = torch.nn.functional.max_pool2d(x, 2)
        x = conv(conv(x))
        skips.append(x)
    for l in range(levels - 2, -1, -1):
        x = conv(conv(torch.cat([skips[l], x.repeat_interleave(2, 2).repeat_interleave(2, 3)], 1)))
    w, b = next(it)
    return (torch.einsum("bchw,oc->bhwo", x, w[:, :, 0, 0]) + b).numpy()


def test_infinite_inputs(ctx):
    import torch
    from paper_2604_03748_amd import lnm

    params = he_normal_params(2, 16, seed=9, bias="uniform")
    g = np.random.default_rng(1).random((1, 24, 40, 3)).astype(np.float32)
    g[0, 5, 7, 0], g[0, 18, 30, 1] = np.inf, -np.inf
    z = torch.empty((1, 24, 40, 6), device="cuda")
    lnm.Net(ctx, 2, 16, params).infer(to_dev(g), logits=z)
    got, ref = to_host(z), _torch_logits(params, 2, 16, g)
    fin = np.isfinite(ref)
    log(f"{(~fin).sum()} logits are not finite")
    assert 0 < (~fin).sum() < ref.size and np.array_equal(fin, np.isfinite(got))
    assert np.array_equal(np.isnan(ref), np.isnan(got)) and np.array_equal(np.isposinf(ref), np.isposinf(got))
    assert np.abs(got[fin] - ref[fin]).max() <= 1e-4 * max(1.0, np.abs(ref[fin]).max())


def test_finite_values_past_bf16(ctx):
    """Activations between bf16's largest number and fp32's: the first layer
    copies the guide scaled to 3.395e38, the second scales back down."""
    import torch
    from paper_2604_03748_amd import lnm

    base, params = 16, he_normal_params(2, 16, seed=9)
    layers, at = unet_layers(2, 16), 0
    for k, (_, ci, co, ks) in enumerate(layers):
        n = co * ci * ks * ks
        w = params[at:at + n].reshape(co, ci, ks, ks)
        if k == 0:  # centre taps: output o copies guide channel o % 3
            w[:] = 0.0
            for o in range(co):
                w[o, o % 3, 1, 1] = 3.395e38
        if k == 1:  # one tap of one input each, so that no partial sum leaves the range
            w[:] = 0.0
            for o in range(co):
                w[o, (5 * o) % ci, o % 3, (o // 3) % 3] = (1.0 + 0.03 * o) * 1e-30
        if k == 2:  # the bottleneck's input is then about 3e8
            w *= 3e-9
        if k == 4:  # and so is the skip half of the decoder's
            w[:, :base] *= 3e-9
        at += n + co
    g = np.random.default_rng(2).random((1, 12, 20, 3)).astype(np.float32)
    g[g > 0.5] = 1.0
    z = torch.empty((1, 12, 20, 6), device="cuda")
    lnm.Net(ctx, 2, 16, params).infer(to_dev(g), logits=z)
    got, ref = to_host(z), _torch_logits(params, 2, 16, g)
    assert np.isfinite(ref).all() and np.abs(ref).max() > 0.1
    err = np.abs(got - ref).max() / np.abs(ref).max()
    log(f"relative error {err:.3g}")
    assert err <= 1e-4
