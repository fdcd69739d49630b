"""Batches of low images, whose layers have enough workgroups for tall tiles but
too few rows to fill them: each image is the same alone (few workgroups, low
tiles) and in the batch, bit for bit, in every precision."""
import numpy as np
import pytest

from synth.weights import he_normal_params
from tests.helpers import log, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp8"])
@pytest.mark.parametrize("levels,base,batch,height,width", [
    (5, 32, 36, 16, 32),   # 16, 8, 4, 2, 1 rows
    (2, 128, 40, 12, 72),  # 12 and 6
    (3, 48, 33, 40, 52),   # 40, 20, 10
])
def test_alone_and_in_a_batch(prec, levels, base, batch, height, width):
    import torch
    from paper_2604_03748_amd import lnm

    ctx = lnm.Context(0)
    params = he_normal_params(levels, base, seed=levels, bias="uniform")
    guide = to_dev(np.random.default_rng(base).random((batch, height, width, 3)))
    code, scales = {"fp32": lnm.FP32, "bf16": lnm.BF16, "fp8": lnm.FP8_E4M3}[prec], None
    if prec == "fp8":
        scales = lnm.Net(ctx, levels, base, params).calibrate_amax(guide[:4].contiguous())
    net = lnm.Net(ctx, levels, base, params, precision=code, act_scales=scales)
    both = net.infer(guide)
    log(f"{prec} {levels} levels, base {base}, {batch} x {height} x {width}: mean {float(both.mean()):.6g}")
    assert torch.isfinite(both).all()
    for b in (0, 1, batch - 1):
        assert torch.equal(both[b], net.infer(guide[b:b + 1].contiguous())[0]), b
