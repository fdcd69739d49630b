"""Reference lightmaps on grids and views where the march's interior part can
go wrong (axes of one to three cells, non-cubic grids, rays along an axis,
views that are no multiple of the pixel tile,
pixels too wide for its boxes), against the fp64 oracle at
the bound of the other reference test."""
import numpy as np
import pytest

from synth.scene import ORTHOGRAPHIC, PERSPECTIVE, Camera
from tests.helpers import log, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,proj,eye,size,step", [
    ((1, 5, 9), PERSPECTIVE, (3.0, 0.7, 0.4), (13, 7), 0.5),
    ((3, 2, 2), ORTHOGRAPHIC, (0.5, 0.5, 3.0), (9, 5), 0.25),
    ((17, 9, 30), ORTHOGRAPHIC, (3.0, 0.5, 0.5), (21, 11), 0.5),
    ((30, 17, 9), PERSPECTIVE, (0.45, 0.5, 0.55), (12, 10), 1.0),  # from inside the volume
    ((8, 8, 1), PERSPECTIVE, (1.5, 2.0, 2.5), (6, 3), 2.0),
    ((90, 70, 101), PERSPECTIVE, (3.0, 0.7, 0.4), (6, 5), 1.0),  # pixels of many voxels: no box fits
    ((40, 48, 64), PERSPECTIVE, (2.3, 1.9, 2.1), (30, 22), 0.5),  # boxes of 8 to 32 steps
])
def test_reference_edges(orc, shape, proj, eye, size, step):
    from paper_2604_03748_amd import lnm

    vol = np.random.default_rng(sum(shape)).random(shape, dtype=np.float32) * 2.0
    target = (0.5, 0.5, 0.5) if eye != (0.45, 0.5, 0.55) else (1.0, 0.6, 0.3)
    cam = Camera(proj, eye, target=target, width=size[0], height=size[1])
    ref = orc.reference_lightmaps(vol, 8.0, cam, step)
    got = to_host(lnm.Context(0).reference_lightmaps(to_dev(vol), 8.0, cam, step))
    d, tol = np.abs(got - ref), 1e-4 * np.abs(ref) + 2e-5
    log(f"reference {shape} {size}: max abs {d.max():.3g}, worst ratio {(d / tol).max():.3g}")
    assert np.all(d <= tol)
