"""The z order on grids of more z cells than sort buckets: the same guiding map
as in band order, and the records spread over the buckets instead of piling up
in the last one."""
import numpy as np
import pytest

from synth.scene import PERSPECTIVE, Camera
from tests.helpers import log, to_dev

pytestmark = pytest.mark.gpu

BUCKETS, HIST = 256, 32  # buckets; their counts' place in the march's counter block (ints)


def _histogram(ws, w, h):
    """The records per bucket that a march left in its workspace: [K][P] fp32
    planes (five), [P] record counts, the counter block, whose first eight
    values sum to the counts."""
    import torch

    up = lambda n: (n + 255) // 256 * 256  # noqa: E731
    for k in range(1, 4096):
        at = 5 * up(4 * k * w * h)
        if at + up(4 * w * h) + 4 * (HIST + BUCKETS) > ws.numel():
            break
        cnt = ws[at:at + 4 * w * h].view(torch.int32).long()
        ctr = ws[at + up(4 * w * h):][:4 * (HIST + BUCKETS)].view(torch.int32).long()
        if cnt.min() >= 0 and cnt.max() <= k and cnt.sum() > 0 and ctr[:8].sum() == cnt.sum():
            return ctr[HIST:].cpu().numpy()
    raise AssertionError("no counter block found")


@pytest.mark.parametrize("given", [False, True])
@pytest.mark.parametrize("nz", [256, 257, 400, 1030])
def test_tall_grids(nz, given):
    import torch
    from paper_2604_03748_amd import lnm

    ctx = lnm.Context(0)
    vol = to_dev(np.random.default_rng(nz).random((nz, 6, 5), dtype=np.float32) * 0.2 + 0.1)
    cam = Camera(PERSPECTIVE, (3.0, 0.6, 0.4), width=64, height=64)
    prm = lnm.make_params(8.0, seed=2, work_order=lnm.ORDER_Z)
    bricks = ctx.make_bricks(vol) if given else None
    ws = torch.zeros(ctx.march_workspace_bytes(vol, 2.0, cam, prm, bricks), dtype=torch.uint8, device="cuda")
    out = ctx.march(vol, 2.0, cam, prm, workspace=ws, bricks=bricks)
    assert torch.equal(out, ctx.march(vol, 2.0, cam, lnm.make_params(8.0, seed=2, work_order=lnm.ORDER_BANDS)))
    hist = _histogram(ws, 64, 64)
    log(f"nz {nz}: {int((hist > 0).sum())} buckets used, the last holds {int(hist[-1])} of {int(hist.sum())}")
    # the samples are spread evenly over z
    assert hist[-1] <= 0.05 * hist.sum()
