"""Exact rays in parts folded on one lane, on the host (hipcc; nothing runs on a
GPU): bit for bit what the parts on a lane each combine to; every tile placed
once in each order; the line between 32- and 64-bit plane offsets."""
import ctypes
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

import inputs
from paper_2206_08660_amd import vdi as V
from tests import synth
from tests.test_split_host import bind

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    # The host half alone: the kernels' code object, which nothing here launches, is left out (its symbol is 0).
    tmp = tmp_path_factory.mktemp("foldhost")
    obj, out = str(tmp / "fold_host.o"), str(tmp / "libfold_host.so")
    subprocess.run(["hipcc", "--offload-arch=gfx950", "--offload-host-only", "-O2", "-std=c++17", "-fPIC", "-c",
                    "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2206_08660_amd", "csrc"),
                    os.path.join(HERE, "host", "fold_host.hip"), "-o", obj], check=True, capture_output=True)
    names = subprocess.run(["nm", "-u", obj], check=True, capture_output=True, text=True).stdout
    fatbin = re.findall(r"__hip_fatbin\w*", names)
    subprocess.run(["hipcc", "-shared", "-fPIC", obj, "-o", out, *("-Wl,--defsym=" + n + "=0" for n in fatbin)], check=True,
                   capture_output=True)
    L = ctypes.CDLL(out)
    P, I = ctypes.c_void_p, ctypes.c_int
    L.host_fold.argtypes = [ctypes.POINTER(V.Desc), P, ctypes.POINTER(V.Camera), I, I, I, I, P, P]
    L.host_tiles_order.argtypes = [I, I, P, I, I, I, I, P]
    L.host_fits32.argtypes = [I, I, I, ctypes.POINTER(ctypes.c_uint64)]
    D = ctypes.POINTER(ctypes.c_double)
    L.host_lists.argtypes = [ctypes.POINTER(V.Desc), P, ctypes.POINTER(V.Camera), I, I, D, D]
    L.host_split_launch.argtypes = [ctypes.c_double, ctypes.c_double]
    return L


# Opacities up to 0.12 (long rays) and up to 0.95 (most rays terminate, in any part).
@pytest.mark.parametrize("alpha_max", [0.12, 0.95])
@pytest.mark.parametrize("theta", [0.0, 4.0, 31.0, -140.0])
@pytest.mark.parametrize("ess", [1, 0])
def test_folded_rays_are_split_rays(host, theta, alpha_max, ess):
    for seed, empty in ((5, 0.1), (6, 0.7)):
        v = synth.random_vdi(31, 22, 24, seed=seed, alpha_max=alpha_max, empty_frac=empty)
        d, grid, _keep = bind(v)
        for W, H in ((38, 26), (31, 23)):
            for parts in (1, 2, 4, 8, 16):
                folded, split = np.zeros((2, H, W, 4), np.float32)
                assert host.host_fold(ctypes.byref(d), grid.ctypes.data, ctypes.byref(V.camera(inputs.orbit_camera(theta))),
                                      W, H, parts, ess, folded.ctypes.data, split.ctypes.data) == 0
                assert np.array_equal(folded, split)


@pytest.mark.parametrize("order", [0, 1, 2])
def test_every_tile_is_placed_once_in_any_order(host, order):
    rng = np.random.default_rng(9)
    sizes = [(1, 260)] * 250 + [(600, 1400)] * 8
    for k, (lo, hi) in enumerate(sizes):
        W, H = (int(x) for x in rng.integers(lo, hi, 2))
        tw, th = (1 << int(x) for x in rng.integers(0 if lo == 1 else 1, 5 if lo == 1 else 4, 2))
        r = np.array([*(rng.integers(0, n + 1) for n in (W, H, W, H))], np.int32)
        if lo > 1 or rng.random() < 0.2:
            r[:] = 0, 0, W, H
        nx, ny = -(-W // tw), -(-H // th)
        placed = np.zeros(nx * ny, np.int32)
        host.host_tiles_order(W, H, r.ctypes.data, tw, th, int(rng.integers(1, 9)), order, placed.ctypes.data)
        assert set(placed) <= {100, 101}, (W, H, r, tw, th)
        x, y = np.meshgrid(np.arange(nx) * tw, np.arange(ny) * th)
        meets = (x < r[2]) & (x + tw > r[0]) & (y < r[3]) & (y + th > r[1]) & (r[2] > r[0]) & (r[3] > r[1])
        assert (placed.reshape(ny, nx)[meets] == 100).all()


def test_offsets_fit_32_bits_up_to_4_gib_of_colours(host):
    o = (ctypes.c_uint64 * 3)()
    seen = set()
    for WO, HO, NS in [(1, 1, 1), (1920, 1080, 50), (1280, 720, 255), (1281, 822, 255), (32768, 8192, 1), (32768, 8190, 1),
                       (32767, 8191, 1), (16384, 16383, 1), (2049, 2047, 64), (2049, 2047, 63), (32768, 32768, 255)]:
        fits = host.host_fits32(WO, HO, NS, o)
        padded = (WO + 1) // 2 * 2 * ((HO + 1) // 2 * 2) * NS
        assert o[2] == padded and fits == (padded * 16 <= 2 ** 32 - 1)
        assert o[1] < padded
        if fits:   # byte offsets of the largest elements, colours, do not wrap
            assert o[0] == o[1] and o[1] * 16 + 15 < 2 ** 32
        seen.add(bool(fits))
    assert seen == {True, False}


def test_launches_that_split_rays(host):
    f = lambda rays, others=0: bool(host.host_split_launch(rays, others))
    assert f(128 * 128) and f(512 * 512) and f(24 * 128 * 128) and f(4 * 256 * 256)
    assert not f(32 * 128 * 128) and not f(8 * 256 * 256)
    # Beside other frames, up to a million rays.
    assert f(4 * 512 * 360, 230_000) and f(850_000, 147_000) and not f(1_600_000, 276_000)
    assert not f(64 * 128 * 128, 10_000_000)


def test_lists_crossed_is_that_of_the_rays(host):
    v = synth.random_vdi(131, 97, 3, seed=12)
    d, grid, _keep = bind(v)
    rng = np.random.default_rng(13)
    most = 0.0
    for k in range(200):
        a, b, rad = rng.uniform(-3, 3), rng.uniform(-1, 1), rng.uniform(0.05, 3.0)
        target = tuple(rng.uniform(-1.0, 1.0, 3)) if k % 2 else (0.0, 0.0, 0.0)
        cam = inputs.Camera(eye=(rad * np.sin(a), rad * b, rad * np.cos(a)), target=target, up=(0.0, 1.0, 0.0),
                            fov_y_deg=float(rng.uniform(20, 120)))
        if k % 20 == 0:
            cam = inputs.orbit_camera(0.5 * k - 20.0)
        got, want = ctypes.c_double(), ctypes.c_double()
        assert host.host_lists(ctypes.byref(d), grid.ctypes.data, ctypes.byref(V.camera(cam)), int(rng.integers(1, 900)),
                               int(rng.integers(1, 900)), ctypes.byref(got), ctypes.byref(want)) == 0
        assert got.value == pytest.approx(want.value, rel=1e-9, abs=1e-9)
        most = max(most, want.value)
    assert most > 50.0
