"""Calls at the edges of what the entry points accept (needs an MI355X): eyes
far from the volume."""
import numpy as np
import pytest

import inputs

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
