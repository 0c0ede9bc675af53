"""Which device planes an upload reads in place, on the host (hipcc; nothing
runs on a GPU): memory of the VDI's own device, aligned to a slot.  Planes of
another device, whose memory need not be mapped, host memory and managed memory
are copied, which the runtime does from anywhere."""
import ctypes
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
HOST, DEVICE, MANAGED, UNREGISTERED = 1, 2, 3, 0   # hipMemoryType


@pytest.fixture(scope="module")
def in_place(tmp_path_factory):
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    out = str(tmp_path_factory.mktemp("planeshost") / "libplanes_host.so")
    cmd = ["hipcc", "--offload-arch=gfx950", "-O1", "-std=c++17", "-fPIC", "-shared",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2206_08660_amd", "csrc"),
           os.path.join(HERE, "host", "planes_host.hip"), "-o", out]
    subprocess.run(cmd, check=True, capture_output=True)
    L = ctypes.CDLL(out)
    L.host_in_place.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_uint64, ctypes.c_int, ctypes.c_uint64]
    return L.host_in_place


def test_only_aligned_memory_of_the_same_device(in_place):
    at = 0x7F0000001000
    for device in (0, 1):
        for plane_device in (0, 1):
            assert in_place(DEVICE, 0, plane_device, at, device, 16) == (device == plane_device)
            for kind in (HOST, MANAGED, UNREGISTERED):
                assert not in_place(kind, 0, plane_device, at, device, 16)
            assert not in_place(DEVICE, 1, plane_device, at, device, 16)
    for align in (1, 8, 16):
        for off in range(0, 32):
            assert in_place(DEVICE, 0, 0, at + off, 0, align) == (off % align == 0)
