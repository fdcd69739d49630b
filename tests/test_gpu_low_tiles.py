"""The bf16 and fp8 convolutions' tiles: an image alone (the small tiles, its
splits in separate workgroups) and in a batch large enough for the tall and
wide ones (and for splits in one workgroup) gives the same lightmaps bit for
bit, at channel counts that leave a block partly empty and image sizes that
are no multiple of the tiles; so does the head in the last layer's epilogue
and as a kernel of its own.  The small tiles are compared with the oracle
elsewhere."""
import numpy as np
import pytest

from synth.weights import he_normal_params
from tests.helpers import log, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2604_03748_amd import lnm

    return lnm.Context(0)


@pytest.mark.parametrize("precision", ["bf16", "fp8"])
@pytest.mark.parametrize("levels,base,B,H,W", [
    (3, 16, 64, 36, 68),   # 16 and 48 input channels in chunks of 32
    (3, 48, 32, 52, 84),   # 48 channels per workgroup, the head over 48
    (2, 80, 24, 66, 50),   # 80 = 64 + 16
    (4, 32, 24, 72, 136),  # splits of the deep levels in one workgroup
])
def test_alone_and_in_a_batch(ctx, precision, levels, base, B, H, W):
    import torch
    from paper_2604_03748_amd import lnm

    params = he_normal_params(levels, base, seed=7, bias="uniform")
    g = to_dev(np.random.default_rng(base + W).random((B, H, W, 3)) * np.array([2.5, 1.0, 3.5]))
    scales = lnm.Net(ctx, levels, base, params).calibrate_amax(g[:1]) if precision == "fp8" else None
    net = lnm.Net(ctx, levels, base, params, precision=lnm.FP8_E4M3 if precision == "fp8" else lnm.BF16,
                  act_scales=scales)
    batch = net.infer(g)
    for k in (0, B - 1):
        alone = net.infer(g[k:k + 1].contiguous())
        assert torch.equal(batch[k], alone[0]), (precision, base, k)
    logits = torch.empty_like(batch)
    separate = net.infer(g, logits=logits)
    log(f"{precision} L{levels}b{base} {B}x{H}x{W}: std {float(batch.std()):.3g}")
    assert torch.equal(separate, batch) and float(batch.std()) > 1e-3
    assert np.isfinite(to_host(logits)).all()
