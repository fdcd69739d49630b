"""Reference lightmaps of a grid with infinite densities: opaque, as densities
far beyond the termination depth are.  Where a sample lies exactly on a grid
line (its weight of the infinite corner is 0, and the product no number) the
value is not defined: of the million samples of these views, whose fractions
take steps of 2^-19 at least, less than one in the mean."""
import numpy as np
import pytest

from synth.scene import ORTHOGRAPHIC, PERSPECTIVE, Camera
from tests.helpers import log, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("proj,width,height,n,what", [
    (PERSPECTIVE, 24, 18, 20, "corners from the LDS box"),
    (ORTHOGRAPHIC, 19, 27, 24, "corners from the LDS box"),
    (PERSPECTIVE, 5, 4, 90, "corners gathered: pixels of many voxels"),
])
def test_infinite_density_is_opaque(proj, width, height, n, what):
    from paper_2604_03748_amd import lnm

    ctx = lnm.Context(0)
    rng = np.random.default_rng(n)
    rho = rng.random((n, n, n), dtype=np.float32) * 0.3
    a, b = int(0.4 * n), int(0.6 * n)
    cam = Camera(proj, (2.31, 1.07, -0.83), width=width, height=height)
    maps = []
    for v in (np.inf, 1e30):
        rho[a:b, a:b, a:b] = v
        maps.append(to_host(ctx.reference_lightmaps(to_dev(rho), 4.0, cam, 0.5)))
    diff = np.sum(~(maps[0] == maps[1]))
    log(f"{what}: {diff} of {maps[0].size} values differ, {np.isnan(maps[0]).sum()} are no numbers")
    assert np.isfinite(maps[1]).all()
    assert diff <= 2
