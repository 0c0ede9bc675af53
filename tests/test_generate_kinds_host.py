"""The instances of the GPU generator's kernel, compiled for the host (hipcc,
no GPU), against the CPU FP64 generator, bit for bit: paired float and uint16
voxels and volumes one voxel wide, sample caches that hold every sample and
that do not, at the cache sizes that vdi_generate allocates."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

import inputs
from paper_2206_08660_amd import vdi as V

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CARD = 256 * 4 * 3 * 64          # lanes of a launch that fills the device
CROWD = (4 << 30) // 16 // 40    # so many that each lane caches 40 samples


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    out = str(tmp_path_factory.mktemp("genkinds") / "libgen_kinds_host.so")
    cmd = ["hipcc", "--offload-arch=gfx950", "-O2", "-std=c++17", "-fPIC", "-shared",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2206_08660_amd", "csrc"),
           os.path.join(HERE, "host", "gen_kinds_host.hip"), "-o", out]
    subprocess.run(cmd, check=True, capture_output=True)
    L = ctypes.CDLL(out)
    P, I = ctypes.c_void_p, ctypes.POINTER(ctypes.c_int)
    L.host_generate_kind.argtypes = [ctypes.POINTER(V.Volume), ctypes.POINTER(V.GenParams), P, P, P, P, ctypes.c_uint64,
                                     I, I, I]
    return L


def check(L, vol, cam, W, H, ns, tf, gamma, lanes, compare=True):
    """Generate on the host, compare with the CPU generator; (cache entries, fits, supersegments)."""
    nz, ny, nx = vol.shape
    bmin, bmax = inputs.aabb_for((nx, ny, nz))
    # Voxels a load must not reach surround the volume: as floats they are NaN.
    flat = np.concatenate([x.view(np.uint8).ravel() for x in (np.full(64, 0xFFFFFFFF, np.uint32), vol,
                                                              np.full(64, 0xFFFFFFFF, np.uint32))])
    v = V.Volume(nx, ny, nz, 1 if vol.dtype == np.uint16 else 0, ctypes.c_void_p(flat.ctypes.data + 256))
    v.aabb_min[:] = bmin
    v.aabb_max[:] = bmax
    p = V.GenParams()
    p.camera_VO = V.camera(cam)
    p.width, p.height, p.max_supersegments, p.tf, p.gamma = W, H, ns, tf, gamma
    count = np.zeros((H, W), np.uint8)
    depth = np.zeros((ns, H, W, 2), np.float32)
    rgba = np.zeros((ns, H, W, 4), np.float32)
    gam = np.zeros((H, W))
    K, fits, over = (ctypes.c_int() for _ in range(3))
    assert L.host_generate_kind(ctypes.byref(v), ctypes.byref(p), count.ctypes.data, depth.ctypes.data, rgba.ctypes.data,
                                gam.ctypes.data, lanes, ctypes.byref(K), ctypes.byref(fits), ctypes.byref(over)) == 0
    assert over.value == 0, f"{over.value} samples written behind a cache of {K.value}"
    if not compare:
        return K.value, bool(fits.value), int(count.sum())
    ref = inputs.generate_vdi(vol, cam, W, H, ns, tf, gamma)
    assert np.array_equal(count, ref.count) and np.array_equal(gam, ref.gamma)
    assert np.array_equal(depth.view(np.uint32), ref.depth.view(np.uint32))
    assert np.array_equal(rgba.view(np.uint32), ref.rgba.view(np.uint32))
    return K.value, bool(fits.value), int(ref.count.sum())


def volume(dims, u16, seed=4):
    nx, ny, nz = dims
    v = np.random.default_rng(seed).random((nz, ny, nx)).astype(np.float32)
    return (v * 65535).astype(np.uint16) if u16 else v


@pytest.mark.parametrize("lanes", [CARD, CROWD])
@pytest.mark.parametrize("u16", [False, True])
@pytest.mark.parametrize("dims", [(48, 40, 33), (2, 61, 5), (1, 9, 47)])
def test_every_instance_matches_the_cpu_generator(host, dims, u16, lanes):
    vol = volume(dims, u16)
    for cam, W, H, ns, tf, gamma in [(inputs.orbit_camera(33.0), 37, 23, 6, inputs.TF_RAMP, 0.0),
                                     (inputs.orbit_camera(-120.0, radius=0.3), 28, 20, 9, inputs.TF_KNOTS4, 0.0),
                                     (inputs.orbit_camera(71.0), 21, 17, 9, inputs.TF_KNOTS4, 0.01)]:
        K, fits, n = check(host, vol, cam, W, H, ns, tf, gamma, lanes)
        assert n > 0 and fits == (lanes == CARD)


@pytest.mark.parametrize("u16", [False, True])
@pytest.mark.parametrize("eye,fov", [(2.0e5, 4e-4), (3.0e9, 2e-8), (1.6e14, 4e-13), (1.5e15, 4e-14), (2.0e15, 4e-14)])
def test_samples_of_far_eyes_stay_in_the_cache(host, eye, fov, u16):
    """The rounding of t1 - t0 grows with the eye's distance and gives rays more samples than the volume's
    diagonal has voxels."""
    vol = volume((32, 32, 32), u16)
    cam = inputs.Camera(eye=(eye, eye, eye), target=(0.0, 0.0, 0.0), up=(0.0, 1.0, 0.0), fov_y_deg=fov)
    _, fits, n = check(host, vol, cam, 25, 21, 5, inputs.TF_KNOTS4, 0.02, CARD, compare=False)
    assert fits and n > 0


@pytest.mark.parametrize("lanes", [CARD, CROWD])
@pytest.mark.parametrize("dims,u16", [((24, 31, 40), False), ((32, 32, 32), True), ((1, 9, 40), False)])
def test_far_eyes_match_the_cpu_generator(host, dims, u16, lanes):
    """Down to where a sample's length and a supersegment's are their ends' rounding: powers of any exponent, and
    distances that the FP32 filter has no bound for."""
    vol, found = volume(dims, u16), 0
    for eye, fov in [(2.0e4, 4e-3), (2.0e6, 4e-5), (3.0e8, 2e-7), (7.0e10, 8e-10), (1.0e13, 7e-12), (1.6e14, 4e-13),
                     (1.5e15, 4e-14)]:
        cam = inputs.Camera(eye=(eye, 0.9 * eye, eye), target=(0.0, 0.0, 0.0), up=(0.0, 1.0, 0.0), fov_y_deg=fov)
        for tf, gamma in [(inputs.TF_KNOTS4, 0.0), (inputs.TF_KNOTS4, 0.02), (inputs.TF_RAMP, 0.0)]:
            _, _, n = check(host, vol, cam, 25, 21, 5, tf, gamma, lanes)
            found += n
    assert found > 100
