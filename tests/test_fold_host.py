"""Exact rays in parts folded on one lane, on the host (hipcc; nothing runs on a
GPU): bit for bit what the parts on a lane each combine to."""
import ctypes
import os
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
    out = str(tmp_path_factory.mktemp("foldhost") / "libfold_host.so")
    cmd = ["hipcc", "--offload-arch=gfx950", "-O2", "-std=c++17", "-fPIC", "-shared",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2206_08660_amd", "csrc"),
           os.path.join(HERE, "host", "fold_host.hip"), "-o", out]
    subprocess.run(cmd, check=True, capture_output=True)
    L = ctypes.CDLL(out)
    P, I = ctypes.c_void_p, ctypes.c_int
    L.host_fold.argtypes = [ctypes.POINTER(V.Desc), P, ctypes.POINTER(V.Camera), I, I, I, I, P, P]
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


def test_launches_that_split_rays(host):
    f = lambda rays, others=0: bool(host.host_split_launch(rays, others))
    assert f(128 * 128) and f(512 * 512) and f(24 * 128 * 128) and f(4 * 256 * 256)
    assert not f(32 * 128 * 128) and not f(8 * 256 * 256)
    # Beside other frames, up to a million rays.
    assert f(4 * 512 * 360, 230_000) and f(850_000, 147_000) and not f(1_600_000, 276_000)
    assert not f(64 * 128 * 128, 10_000_000)
