"""z order with the caller's bricks and room for the plane pairs: whether the
grid holds enough density to repay the pairs' copy is found out on the device,
and the map equals the band order's either way."""
import numpy as np
import pytest

from synth.scene import ORTHOGRAPHIC, PERSPECTIVE, Camera
from tests.helpers import log, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(40, 40, 40), (300, 13, 22)])
@pytest.mark.parametrize("fill", ["all", "corner", "none"])
@pytest.mark.parametrize("proj", [PERSPECTIVE, ORTHOGRAPHIC])
def test_full_and_nearly_empty_grids(shape, fill, proj):
    import torch
    from paper_2604_03748_amd import lnm

    ctx = lnm.Context(0)
    rho = np.random.default_rng(5).random(shape, dtype=np.float32)
    if fill != "all":
        rho[4:] = 0.0
        rho[:, 4:] = 0.0
        rho[:, :, 4 if fill == "corner" else 0:] = 0.0
    vol = to_dev(rho)
    bricks = ctx.make_bricks(vol)
    cam = Camera(proj, (2.6, 0.9, -0.4), width=67, height=61)
    maps = {}
    for order in (lnm.ORDER_Z, lnm.ORDER_BANDS):
        prm = lnm.make_params(0.7 * max(shape) / 40, seed=3, work_order=order)
        if order == lnm.ORDER_Z:  # room for the pairs is asked for
            assert ctx.march_workspace_bytes(vol, 8.0, cam, prm, bricks) == ctx.march_workspace_bytes(vol, 8.0, cam, prm)
        maps[order] = ctx.march(vol, 8.0, cam, prm, bricks=bricks)
    log(f"{shape} {fill}: guide sum {float(maps[lnm.ORDER_Z].sum()):.6g}")
    assert torch.equal(maps[lnm.ORDER_Z], maps[lnm.ORDER_BANDS])
