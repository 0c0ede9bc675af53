"""The ray walkers' arithmetic of bounds on the host (hipcc; nothing runs on a
GPU): the largest float at or below a depth and the smallest at or above it, for
depths of either sign, and the clipping of a ray's parameter range against
IEEE division, up to quotients beyond the double range."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    out = str(tmp_path_factory.mktemp("boundshost") / "libbounds_host.so")
    cmd = ["hipcc", "--offload-arch=gfx950", "-O2", "-std=c++17", "-fPIC", "-shared",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2206_08660_amd", "csrc"),
           os.path.join(HERE, "host", "bounds_host.hip"), "-o", out]
    subprocess.run(cmd, check=True, capture_output=True)
    return ctypes.CDLL(out)


def p(a):
    return ctypes.c_void_p(a.ctypes.data)


def test_floats_next_to_a_depth(host):
    rng = np.random.default_rng(3)
    f = np.concatenate((rng.random(500) * 10.0 ** rng.integers(-44, 38, 500), [0.0, 1.4e-45, 3.4028234e38])).astype(np.float32)
    f = np.concatenate((f, -f))
    z = f.astype(np.float64)
    z = np.concatenate((z, np.nextafter(z, np.inf), np.nextafter(z, -np.inf), z * (1 + 3e-9), z * (1 - 3e-9),
                        [1e-50, -1e-50, 1e-300, -1e-300, 0.0, -0.0]))
    below, above = np.zeros((2, len(z)), np.float32)
    host.host_float_bounds(p(z), len(z), p(below), p(above))
    with np.errstate(over="ignore"):
        near = z.astype(np.float32)
        down = np.where(near.astype(np.float64) > z, np.nextafter(near, np.float32(-np.inf)), near)
        up = np.where(near.astype(np.float64) < z, np.nextafter(near, np.float32(np.inf)), near)
    assert np.array_equal(below, down) and np.array_equal(above, up)


def test_clip_is_a_division(host):
    rng = np.random.default_rng(4)
    a = np.concatenate(([0.0], 10.0 ** rng.uniform(-30, 38, 200)))
    b = np.concatenate(([0.0], 10.0 ** rng.uniform(-299.9, 3, 200), 10.0 ** rng.uniform(-5, 1, 100)))
    a, b = (x.ravel() for x in np.meshgrid(np.concatenate((a, -a)), np.concatenate((b, -b))))
    lo, hi = np.zeros(len(a)), np.full(len(a), np.inf)
    ok = np.zeros(len(a), np.int32)
    host.host_clip(p(a), p(b), len(a), p(lo), p(hi), p(ok))
    with np.errstate(all="ignore"):
        t = -a / b
    want_lo, want_hi = np.where(b > 0, np.maximum(0.0, t), 0.0), np.where(b < 0, np.minimum(np.inf, t), np.inf)
    empty = np.where(b == 0, a < 0, ~(want_hi > want_lo))
    assert np.isinf(t[b != 0]).sum() > 100
    assert np.array_equal((ok == 0) | ~(hi > lo), empty)
    live = ~empty
    with np.errstate(invalid="ignore"):
        for got, want in ((lo[live], want_lo[live]), (hi[live], want_hi[live])):
            assert ((got == want) | (np.abs(got - want) <= 4e-16 * np.abs(want))).all()
