"""Views of more than 1024 tiles, whose bands are cut at runs of tiles, and of
131072 pixels and more, whose cell order is sorted by larger blocks: the same
guiding map bit for bit in every order."""
import numpy as np
import pytest

from synth.scene import ORTHOGRAPHIC, PERSPECTIVE, Camera
from tests.helpers import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("proj,size,off_axis", [(PERSPECTIVE, (417, 315), False), (ORTHOGRAPHIC, (369, 356), False),
                                                (PERSPECTIVE, (600, 120), True), (PERSPECTIVE, (1100, 9), False)])
def test_orders_agree(proj, size, off_axis):
    import torch
    from paper_2604_03748_amd import lnm

    ctx = lnm.Context(0)
    vol = to_dev(np.random.default_rng(3).random((40, 37, 44), dtype=np.float32))
    # off axis: the volume in a corner of the view, most tiles empty
    cam = Camera(proj, (2.6, 1.1, 1.4), target=(1.3, 0.9, 0.2) if off_axis else (0.5, 0.5, 0.5), width=size[0],
                 height=size[1])
    maps = [ctx.march(vol, 8.0, cam, lnm.make_params(1.0, seed=5, work_order=o))
            for o in (lnm.ORDER_BANDS, lnm.ORDER_Z, lnm.ORDER_CELLS)]
    assert float(maps[0][..., 0].max()) > 0.0
    assert torch.equal(maps[0], maps[1]) and torch.equal(maps[0], maps[2])
