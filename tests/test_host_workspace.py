"""Workspace sizes on the CPU: the library's host code built with g++ against
the counting launch stubs (tests/hostbuild/fake_device.cpp)."""
import ctypes as C
import os
import shutil
import subprocess

import pytest

from paper_2604_03748_amd import lnm
from synth.weights import n_params

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HB = os.path.join(ROOT, "tests", "hostbuild")
CSRC = os.path.join(ROOT, "paper_2604_03748_amd", "csrc")
ANY = 0x1000  # a device address that is never read

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("host") / "libhost.so")
    sources = [os.path.join(CSRC, f) for f in ("api.hip", "plan.hip", "train_api.hip", "frame_static.hip")]
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", f"-I{HB}", f"-I{os.path.join(ROOT, 'include')}",
                        f"-I{CSRC}", "-x", "c++", *sources, "-x", "none", os.path.join(HB, "fake_device.cpp"), "-o", so],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    L = C.CDLL(so)
    vp, sz = C.c_void_p, C.c_size_t
    for name in ("lnm_march_workspace_bytes", "lnm_march_least_workspace_bytes", "lnm_net_device_bytes",
                 "lnm_frame_workspace_bytes"):
        getattr(L, name).restype = sz
    L.lnm_frame_workspace_bytes.argtypes = [vp, vp, vp, vp]
    L.lnm_frame_static.argtypes = [vp, vp, vp, vp, vp, vp, C.c_int32, vp, vp, vp, vp]
    L.lnm_last_error.restype = C.c_char_p
    return L


@pytest.fixture(scope="module")
def net(host):
    """A context and a base-16 network of the host build."""
    ctx, handle = C.c_void_p(), C.c_void_p()
    assert host.lnm_ctx_create(0, C.byref(ctx)) == 0
    n, bytes_ = n_params(3, 16), host.lnm_net_device_bytes(3, 16, lnm.FP32)
    params = (C.c_float * n)()
    buf = C.create_string_buffer(bytes_ + 256)
    at = (C.addressof(buf) + 255) // 256 * 256
    assert host.lnm_net_create(ctx, 3, 16, lnm.FP32, params, C.c_size_t(n), None, C.c_void_p(at), C.c_size_t(bytes_),
                               None, C.byref(handle)) == 0
    yield ctx, handle
    host.lnm_net_destroy(handle)
    host.lnm_ctx_destroy(ctx)
    del buf


def volume(n, bricks):
    v = lnm.Volume()
    v.density, v.sigma_scale, v.bricks = ANY, 8.0, ANY if bricks else None
    v.nx, v.ny, v.nz = (n, n, n) if isinstance(n, int) else n
    return v


def camera(w, h, ortho=False):
    c = lnm.Camera()
    c.projection = lnm.ORTHOGRAPHIC if ortho else lnm.PERSPECTIVE
    c.eye[:], c.target[:], c.up[:] = (3.0, 0.5, 0.5), (0.5, 0.5, 0.5), (0.0, 1.0, 0.0)
    c.fov_y_deg, c.ortho_half_extent, c.width, c.height = 60.0, 0.8, w, h
    return c


@pytest.mark.parametrize("n,w,h,step", [(192, 192, 192, 4.0), (160, 208, 208, 4.0), (240, 168, 168, 4.0),
                                        (256, 184, 184, 8.0), (192, 256, 128, 4.0)])
def test_static_frame_without_the_optional_copy(host, net, n, w, h, step):
    """Frames in z order whose march fits the static workspace on the caller's
    bricks, but not with the plane pairs beside them, run."""
    ctx, handle = net
    prm = lnm.make_params(step)
    v, c = volume(n, True), camera(w, h)
    st = host.lnm_frame_static(ctx, handle, C.byref(v), C.byref(c), C.byref(prm), None, 0, ANY, ANY, None, None)
    assert st == 0, host.lnm_last_error()


def test_static_frame_beyond_the_workspace(host, net):
    ctx, handle = net
    prm = lnm.make_params(4.0)
    v, c = volume(256, True), camera(512, 512)
    st = host.lnm_frame_static(ctx, handle, C.byref(v), C.byref(c), C.byref(prm), None, 0, ANY, ANY, None, None)
    assert st == lnm.LNM_ERR_SHAPE and b"static workspace" in host.lnm_last_error()


@pytest.mark.parametrize("n,w,h,step,ortho,pairs", [
    (217, 298, 77, 4.0, False, False),   # a wide view: the grid fills a tenth of its pixels
    (160, 125, 236, 8.0, True, False),   # short marches
    ((252, 247, 192), 326, 111, 8.0, False, False),
    (256, 512, 512, 4.0, False, True),
    (224, 365, 445, 4.0, False, True),
])
def test_plane_pairs_beside_bricks(host, n, w, h, step, ortho, pairs):
    """Beside the caller's bricks the march asks for room for the plane pairs
    only where its samples can repay their copy."""
    prm = lnm.make_params(step, work_order=lnm.ORDER_Z)
    c = camera(w, h, ortho)
    own, given = volume(n, False), volume(n, True)
    a, b = (host.lnm_march_workspace_bytes(C.byref(v), C.byref(c), C.byref(prm)) for v in (own, given))
    copy = (8 * (own.nx + 2) * (own.ny + 2) * (own.nz + 1) + 255) // 256 * 256
    assert a - b == (0 if pairs else copy)


@pytest.mark.parametrize("bricks", [False, True])
@pytest.mark.parametrize("n,w,h,step,order", [
    (256, 512, 512, 4.0, lnm.ORDER_AUTO), (192, 64, 64, 4.0, lnm.ORDER_AUTO), (16, 65, 41, 2.0, lnm.ORDER_AUTO),
    (128, 256, 256, 4.0, lnm.ORDER_AUTO), (64, 31, 77, 3.0, lnm.ORDER_BANDS), ((9, 40, 22), 50, 50, 0.7, lnm.ORDER_Z),
])
def test_least_workspace_is_accepted(host, net, n, w, h, step, order, bricks):
    """The march takes its least workspace and refuses one byte less; the
    preferred size is no smaller."""
    ctx, _ = net
    host.lnm_march.argtypes = [C.c_void_p] * 4 + [C.c_void_p, C.c_void_p, C.c_size_t, C.c_void_p]
    prm = lnm.make_params(step, work_order=order)
    v, c = volume(n, bricks), camera(w, h)
    least, full = (f(C.byref(v), C.byref(c), C.byref(prm)) for f in
                   (host.lnm_march_least_workspace_bytes, host.lnm_march_workspace_bytes))
    assert 0 < least <= full
    for size, want in ((least, 0), (least - 1, lnm.LNM_ERR_SHAPE), (full, 0), (full - 1, 0 if least < full else lnm.LNM_ERR_SHAPE)):
        assert host.lnm_march(ctx, C.byref(v), C.byref(c), C.byref(prm), ANY, ANY, size, None) == want


@pytest.mark.parametrize("n,w,h,step,cells", [
    (32, 64, 64, 2.0, False),                # 16 steps, a small view
    ((24, 48, 192), 348, 1080, 10.0, True),  # 19 steps, a large one
    (64, 874, 693, 3.5, True),               # 18 steps
    (128, 512, 512, 10.0, False),            # 13 steps
    (128, 256, 256, 4.0, True),              # 32 steps
])
def test_order_of_short_marches(host, n, w, h, step, cells):
    """The automatic order of short light marches, by the workspace it asks for."""
    v, c = volume(n, False), camera(w, h)
    size = {o: host.lnm_march_workspace_bytes(C.byref(v), C.byref(c), C.byref(lnm.make_params(step, work_order=o)))
            for o in (lnm.ORDER_AUTO, lnm.ORDER_BANDS, lnm.ORDER_CELLS)}
    assert size[lnm.ORDER_BANDS] != size[lnm.ORDER_CELLS]
    assert size[lnm.ORDER_AUTO] == size[lnm.ORDER_CELLS if cells else lnm.ORDER_BANDS]
