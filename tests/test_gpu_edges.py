"""Calls at the edges of what the entry points accept (needs an MI355X): eyes
far from the volume; device planes that are not memory of the device or not
aligned to a slot, or are still being written on the null stream."""
import ctypes

import numpy as np
import pytest

import inputs
from tests import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    torch.cuda.set_device(0)
    yield
    torch.cuda.synchronize()


def _V():
    from paper_2206_08660_amd import vdi as V
    return V


def on_device(vol):
    return torch.from_numpy(vol.view(np.int16) if vol.dtype == np.uint16 else vol).cuda()


# The last three lie beyond 1e8 samples, where lengths are mostly the rounding of their ends.
@pytest.mark.parametrize("eye,fov", [(2.0e4, 4e-3), (2.0e6, 4e-5), (7.0e10, 8e-10), (1.6e14, 4e-13)])
@pytest.mark.parametrize("u16", [False, True])
def test_far_eyes(eye, fov, u16):
    V = _V()
    vol = np.random.default_rng(4).random((40, 31, 24)).astype(np.float32)
    vol = (vol * 65535).astype(np.uint16) if u16 else vol
    bmin, bmax = inputs.aabb_for((24, 31, 40))
    cam = inputs.Camera(eye=(eye, 0.9 * eye, eye), target=(0.0, 0.0, 0.0), up=(0.0, 1.0, 0.0), fov_y_deg=fov)
    for gamma in (0.0, 0.02):
        ref = inputs.generate_vdi(vol, cam, 25, 21, 5, inputs.TF_KNOTS4, gamma)
        got = V.generate(on_device(vol), bmin, bmax, cam, 25, 21, 5, tf="knots4", gamma=gamma)
        torch.cuda.synchronize()
        print(f"[gpu] eye {eye} gamma {gamma}: {int(ref.count.sum())} supersegments", flush=True)
        for a, b in zip(got, (ref.count, ref.depth, ref.rgba, ref.gamma)):
            assert np.array_equal(a.cpu().numpy(), b)
    f64 = V.dvr(on_device(vol), bmin, bmax, cam, 25, 21, tf="knots4", precision="f64").cpu().numpy()
    assert np.array_equal(f64, ref.dvr.astype(np.float32))


def created(V, d):
    """A Vdi made from the descriptor d as it stands, by the C entry point alone."""
    h = ctypes.c_void_p()
    V._check(V.lib().vdi_create(ctypes.byref(d), ctypes.byref(h)))
    v = V.Vdi.__new__(V.Vdi)
    v._h = h
    v.width, v.height, v.ns, v.store = d.width, d.height, d.max_supersegments, "f32"
    return v


def device_vdi(V, v):
    return V.DeviceVDI(*(torch.from_numpy(a).cuda() for a in (v.count, v.depth, v.rgba)), v.camera, v.bmin, v.bmax,
                       v.grid_k, v.grid_nz, v.grid_z)


@pytest.mark.parametrize("how", ["pinned", "off by 4 bytes"])
def test_planes_not_read_in_place(how):
    """Copied to the device first: pinned host memory, and planes 4 bytes off their slots' alignment."""
    V = _V()
    v = synth.random_vdi(65, 33, 17, seed=82, alpha_max=0.3)
    cam = inputs.orbit_camera(12.0)
    dv = device_vdi(V, v)
    if how == "pinned":
        planes = [torch.from_numpy(a).pin_memory() for a in (v.count, v.depth, v.rgba)]
        ptrs = [t.data_ptr() for t in planes]
    else:
        planes = [torch.cat((torch.zeros(4 // a.itemsize, dtype=torch.from_numpy(a).dtype), torch.from_numpy(a).reshape(-1))).cuda()
                  for a in (v.count, v.depth, v.rgba)]
        ptrs = [t.data_ptr() + 4 for t in planes]
    torch.cuda.synchronize()
    d, _keep = V._desc(dv, "f32", False, None, "f32")
    d.count, d.depth, d.rgba = ptrs
    with V.Vdi(v) as a, created(V, d) as b:
        assert np.array_equal(b.grid(), a.grid()) and b.info().supersegments == int(v.count.sum())
        want = a.render(cam, 60, 44)
        assert torch.equal(b.render(cam, 60, 44), want)
        V._check(V.lib().vdi_replace_begin(b.handle, ctypes.byref(d), None))
        while not b.replace_poll():
            pass
        assert torch.equal(b.render(cam, 60, 44), want)


def test_planes_still_being_written_on_the_null_stream():
    """vdi_create's own stream runs beside the null stream: it waits for it before it reads the planes."""
    V = _V()
    v = synth.random_vdi(200, 120, 20, seed=83, alpha_max=0.3)
    full = device_vdi(V, v)
    late = V.DeviceVDI(*(torch.zeros_like(t) for t in (full.count, full.depth, full.rgba)), v.camera, v.bmin, v.bmax,
                       v.grid_k, v.grid_nz, v.grid_z)
    d, _keep = V._desc(late, "f32", False, None, "f32")
    busy = torch.rand((4096, 4096), device="cuda")
    torch.cuda.synchronize()
    assert torch.cuda.current_stream().cuda_stream == 0
    for _ in range(40):
        torch.mm(busy, busy)
    for a, b in zip((late.count, late.depth, late.rgba), (full.count, full.depth, full.rgba)):
        a.copy_(b)
    cam = inputs.orbit_camera(12.0)
    with created(V, d) as b, V.Vdi(v) as a:
        assert b.info().supersegments == int(v.count.sum())
        assert torch.equal(b.render(cam, 60, 44), a.render(cam, 60, 44))
