"""The z order's plane pairs against its bricks: the same guiding map bit for
bit on the same camera, whichever a workspace has room for and whether or not
the caller gives bricks, on ragged grids, views along z (whose lights leave
their plane), both light sets and an eye inside the volume; and a workspace
of the size that the bricks need is still accepted."""
import numpy as np
import pytest

from synth.scene import ORTHOGRAPHIC, PERSPECTIVE, Camera
from tests.helpers import log, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,proj,eye,light_set", [
    ((9, 22, 35), PERSPECTIVE, (3.0, 0.7, 0.4), 0),
    ((31, 18, 7), PERSPECTIVE, (0.5, 0.5, 3.0), 0),   # along z
    ((16, 16, 16), ORTHOGRAPHIC, (0.5, 0.5, 3.0), 1),
    ((20, 33, 12), PERSPECTIVE, (0.4, 0.5, 0.6), 1),  # from inside
    ((1, 2, 3), ORTHOGRAPHIC, (3.0, 0.5, 0.5), 0),
])
def test_pairs_equal_bricks(shape, proj, eye, light_set):
    import torch
    from paper_2604_03748_amd import lnm

    ctx = lnm.Context(0)
    vol = to_dev(np.random.default_rng(sum(shape)).random(shape, dtype=np.float32) * 1.5)
    target = (0.5, 0.5, 0.5) if eye != (0.4, 0.5, 0.6) else (1.0, 0.6, 0.2)
    cam = Camera(proj, eye, target=target, width=45, height=27)
    prm = lnm.make_params(0.7, seed=3, light_set=light_set, work_order=lnm.ORDER_Z)
    bricks = ctx.make_bricks(vol)
    nz, ny, nx = shape
    up = lambda n: (n + 255) // 256 * 256  # noqa: E731
    pair_b, brick_b = up(8 * (nx + 2) * (ny + 2) * (nz + 1)), up(bricks.numel() * 4)
    big = ctx.march_workspace_bytes(vol, 8.0, cam, prm, bricks)
    assert ctx.march_workspace_bytes(vol, 8.0, cam, prm) == big  # pairs either way
    ws = torch.empty(big + brick_b, dtype=torch.uint8, device="cuda")

    def run(n, br):
        out = torch.empty((27, 45, 3), device="cuda")
        return ctx.march(vol, 8.0, cam, prm, out=out, workspace=ws[:n], bricks=br)

    pairs, given = run(big, None), run(big, bricks)
    own = run(big - pair_b, bricks)  # room for neither: the caller's bricks
    log(f"pairs {shape}: guide sum {float(pairs.sum()):.6g}")
    assert torch.equal(pairs, given) and torch.equal(pairs, own)
    if brick_b < pair_b:
        assert torch.equal(pairs, run(big - pair_b + brick_b, None))  # room for the bricks only
    with pytest.raises(lnm.LnmError):
        run(big - pair_b - 256, bricks)
    bands = ctx.march(vol, 8.0, cam, lnm.make_params(0.7, seed=3, light_set=light_set, work_order=lnm.ORDER_BANDS))
    assert torch.equal(pairs, bands)


def test_short_marches_take_bands():
    """Automatic order at 8 steps per axis: the cells' and the bands' map, also
    in a workspace of the cells' size only."""
    import torch
    from paper_2604_03748_amd import lnm

    ctx = lnm.Context(0)
    vol = to_dev(np.random.default_rng(4).random((16, 16, 16), dtype=np.float32) * 1.5)
    cam = Camera(PERSPECTIVE, (2.5, 0.7, 0.4), width=65, height=41)
    out = {}
    for order in (lnm.ORDER_AUTO, lnm.ORDER_CELLS, lnm.ORDER_BANDS):
        prm = lnm.make_params(2.0, seed=3, work_order=order)
        out[order] = (ctx.march(vol, 8.0, cam, prm).clone(), ctx.march_workspace_bytes(vol, 8.0, cam, prm))
    auto, n_auto = out[lnm.ORDER_AUTO]
    assert n_auto == out[lnm.ORDER_BANDS][1]
    assert torch.equal(auto, out[lnm.ORDER_CELLS][0]) and torch.equal(auto, out[lnm.ORDER_BANDS][0])
    ws = torch.empty(out[lnm.ORDER_CELLS][1], dtype=torch.uint8, device="cuda")
    assert torch.equal(auto, ctx.march(vol, 8.0, cam, lnm.make_params(2.0, seed=3), workspace=ws))
