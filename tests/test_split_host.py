"""How an exact frame is dealt out, on the host (hipcc; nothing runs on a GPU):
rays split into 1 to 16 parts against whole rays and the FP64 oracle, with 32-
and 64-bit plane offsets; the order of a frame's tiles; the bounds of the
volume's box on the image."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

import inputs
import oracle
from paper_2206_08660_amd import vdi as V
from tests import synth
from tests.gpu_util import TOL

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    out = str(tmp_path_factory.mktemp("splithost") / "libsplit_host.so")
    cmd = ["hipcc", "--offload-arch=gfx950", "-O2", "-std=c++17", "-fPIC", "-shared",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2206_08660_amd", "csrc"),
           os.path.join(HERE, "host", "split_host.hip"), "-o", out]
    subprocess.run(cmd, check=True, capture_output=True)
    L = ctypes.CDLL(out)
    P, I = ctypes.c_void_p, ctypes.c_int
    L.host_split.argtypes = [ctypes.POINTER(V.Desc), P, ctypes.POINTER(V.Camera), I, I, I, I, P, ctypes.POINTER(I)]
    L.host_bounds.argtypes = [ctypes.POINTER(V.Desc), P, ctypes.POINTER(V.Camera), I, I, ctypes.POINTER(I)]
    L.host_tiles.argtypes = [I, I, P, I, I, I, P]
    return L


def bind(src):
    d, keep = V._desc(src, "f32", False, None, "f32")
    grid = np.ascontiguousarray(oracle.count_grid(src), dtype=np.uint32)
    gz = np.ascontiguousarray(src.grid_z, dtype=np.float32)
    d.grid_z = gz.ctypes.data
    return d, grid, (keep, gz)


def split(L, src, cam, W, H, parts, wide=False):
    d, grid, _keep = bind(src)
    out, chosen = np.zeros((H, W, 4), np.float32), ctypes.c_int()
    assert L.host_split(ctypes.byref(d), grid.ctypes.data, ctypes.byref(V.camera(cam)), W, H, parts, int(wide),
                        out.ctypes.data, ctypes.byref(chosen)) == 0
    return out, chosen.value


# Opacities up to 0.12 (long rays) and up to 0.95 (most rays terminate).
@pytest.mark.parametrize("alpha_max", [0.12, 0.95])
@pytest.mark.parametrize("theta", [0.0, 4.0, 31.0, -140.0])
def test_split_rays(host, theta, alpha_max):
    v = synth.random_vdi(31, 22, 24, seed=5, alpha_max=alpha_max, empty_frac=0.1)
    cam = inputs.orbit_camera(theta)
    ref = oracle.render_exact(v, cam, 38, 26)
    whole, chosen = split(host, v, cam, 38, 26, 1)
    assert chosen in (1, 2, 4, 8, 16) and (theta != 0.0 or chosen == 1)
    assert np.abs(whole - ref).max() <= TOL
    for parts in (2, 4, 8, 16):
        img, _ = split(host, v, cam, 38, 26, parts)
        wide, _ = split(host, v, cam, 38, 26, parts, wide=True)
        assert np.array_equal(img, wide)
        # Rounding only: a supersegment cut in two, partial products in another
        # order, over at most some hundred pieces of 6e-8 each.  (A product one
        # rounding from the termination limit may stop a piece earlier: 1e-5.)
        assert np.abs(img - whole).max() <= 2e-5
        assert np.abs(img - ref).max() <= TOL


def test_every_tile_is_placed_once(host):
    rng = np.random.default_rng(7)
    for _ in range(400):
        W, H = (int(x) for x in rng.integers(1, 260, 2))
        tw, th = (1 << int(x) for x in rng.integers(0, 5, 2))
        r = np.array([*(rng.integers(0, n + 1) for n in (W, H, W, H))], np.int32)
        if rng.random() < 0.2:
            r[:] = 0, 0, W, H
        nx, ny = -(-W // tw), -(-H // th)
        placed = np.zeros(nx * ny, np.int32)
        host.host_tiles(W, H, r.ctypes.data, tw, th, int(rng.integers(1, 4)), placed.ctypes.data)
        assert set(placed) <= {100, 101}, (W, H, r, tw, th)
        x, y = np.meshgrid(np.arange(nx) * tw, np.arange(ny) * th)
        meets = (x < r[2]) & (x + tw > r[0]) & (y < r[3]) & (y + th > r[1]) & (r[2] > r[0]) & (r[3] > r[1])
        assert (placed.reshape(ny, nx)[meets] == 100).all()


def test_rays_off_the_bounds_miss_the_box(host):
    tiny = inputs.load_workload("tiny", keep_dvr=False)
    rng = np.random.default_rng(11)
    smaller = 0
    for k in range(60):
        a, b, rad = rng.uniform(-3, 3), rng.uniform(-1, 1), rng.uniform(0.2, 3.0)
        eye = (rad * np.sin(a), rad * b, rad * np.cos(a))
        target = tuple(rng.uniform(-1.0, 1.0, 3)) if k % 2 else (0.0, 0.0, 0.0)
        cam = inputs.Camera(eye=eye, target=target, up=(0.0, 1.0, 0.0), fov_y_deg=float(rng.uniform(20, 120)))
        d, grid, _keep = bind(tiny)
        W, H = (int(x) for x in rng.integers(1, 90, 2))
        inside = ctypes.c_int()
        assert host.host_bounds(ctypes.byref(d), grid.ctypes.data, ctypes.byref(V.camera(cam)), W, H,
                                ctypes.byref(inside)) == 0
        smaller += inside.value < W * H
    assert smaller > 20
