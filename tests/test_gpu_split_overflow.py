"""fp32 networks whose sums pass fp32's range: infinite as fp32's own, so that
positive weights end in lightmaps of 1 (a sum of bf16 pieces that overflows
must not become NaN, which the ReLU would turn into 0)."""
import numpy as np
import pytest

from synth.weights import n_params, unet_layers
from tests.helpers import log, to_dev, to_host

pytestmark = pytest.mark.gpu


# 3.3e4 is no bf16 number, nor is 1.1e30: all pieces take part.  Tiles of 4, 8
# and 16 rows, split and unsplit sums.
@pytest.mark.parametrize("levels,base,batch,height,width", [(2, 16, 1, 6, 10), (3, 32, 2, 64, 96), (2, 48, 16, 128, 128)])
def test_overflowing_sums_are_infinite(levels, base, batch, height, width):
    from paper_2604_03748_amd import lnm

    ctx = lnm.Context(0)
    params, at = np.full(n_params(levels, base), 3.3e4, dtype=np.float32), 0
    for _, ci, co, k in unet_layers(levels, base):
        at += co * ci * k * k
        params[at:at + co] = 0.0  # the biases
        at += co
    net = lnm.Net(ctx, levels, base, params)
    guide = to_dev(np.full((batch, height, width, 3), 1.1e30, dtype=np.float32))
    lm = to_host(net.infer(guide))
    log(f"levels {levels} base {base}: lightmaps {lm.min()} .. {lm.max()}")
    assert (lm == 1.0).all()
