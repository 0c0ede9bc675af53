"""The GPU kernels at the sizes where a tile, a split or a special path begins
or ends (needs an MI355X): split exact frames of opaque and thin VDIs, views
that put the volume's box off the image, uploads of ragged VDIs from device
planes, volumes one to three voxels wide, SSIM tiles."""
import numpy as np
import pytest

import inputs
import oracle
from oracle import quality as Q
from tests import synth
from tests.gpu_util import TOL

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


def render(h, cam, W, H, **kw):
    img = h.render(cam, W, H, **kw)
    torch.cuda.synchronize()
    return img.cpu().numpy()


# Frames of 16 lanes a ray down to whole rays; most rays terminate at 0.95.
@pytest.mark.parametrize("alpha_max", [0.12, 0.95])
@pytest.mark.parametrize("W,H", [(1, 1), (5, 3), (64, 48), (150, 101), (301, 211), (640, 411)])
def test_split_frames(W, H, alpha_max):
    v = synth.random_vdi(61, 43, 24, seed=8, alpha_max=alpha_max, empty_frac=0.1)
    with _V().Vdi(v) as h:
        for theta in (0.0, 6.0, 38.0, -130.0):
            cam = inputs.orbit_camera(theta)
            ref, ties = oracle.render_exact(v, cam, W, H, flags=True)
            img = render(h, cam, W, H)
            print(f"[gpu] split {W}x{H} {theta} alpha {alpha_max}", flush=True)
            assert np.abs(img - ref)[ties == 0].max(initial=0.0) <= TOL
            for search in ("seeded", "binary", "linear"):
                assert np.array_equal(render(h, cam, W, H, search=search), img)
            count_img = h.render_counters(cam, W, H)[0]
            torch.cuda.synchronize()
            assert np.array_equal(count_img.cpu().numpy(), img)


@pytest.mark.parametrize("eye,target,fov", [((0.0, 0.0, 1.5), (1.3, 0.2, 0.0), 50.0), ((0.2, 0.1, 0.3), (0.0, 0.0, 0.0), 70.0),
                                            ((0.0, 0.0, 1.5), (0.0, 0.0, 3.0), 50.0), ((0.7, 0.9, 1.4), (0.0, 0.0, 0.0), 20.0)])
@pytest.mark.parametrize("W,H,d_i", [(77, 53, 1.0), (640, 360, 1.0), (640, 360, 4.0)])
def test_box_off_the_image(eye, target, fov, W, H, d_i):
    tiny = inputs.load_workload("tiny", keep_dvr=False)
    cam = inputs.Camera(eye=eye, target=target, up=(0.0, 1.0, 0.0), fov_y_deg=fov)
    with _V().Vdi(tiny) as h:
        img = render(h, cam, W, H, d_i=d_i)
        ref, flags = oracle.render(tiny, cam, W, H, d_i, 0.0)
        assert np.abs(img - ref)[flags == 0].max(initial=0.0) <= TOL
        out = torch.full((H, W, 4), -1.0, dtype=torch.float32, device="cuda")
        h.render(cam, W, H, d_i=2.0, d_r=2.0, out=out)
        torch.cuda.synchronize()
        assert float(out.min()) >= 0.0   # every pixel written


@pytest.mark.parametrize("w,hh,ns", [(1, 1, 1), (2, 3, 9), (63, 5, 8), (64, 2, 7), (65, 33, 17), (130, 1, 255)])
def test_upload_of_ragged_device_planes(w, hh, ns):
    V = _V()
    v = synth.random_vdi(w, hh, ns, seed=w + ns, alpha_max=0.3)
    d = V.DeviceVDI(*(torch.from_numpy(a).cuda() for a in (v.count, v.depth, v.rgba)), v.camera, v.bmin, v.bmax,
                    v.grid_k, v.grid_nz, v.grid_z)
    cam = inputs.orbit_camera(12.0)
    for store in ("f32", "f16", "bf16"):
        with V.Vdi(v, store=store) as a, V.Vdi(d, store=store) as b:
            assert np.array_equal(a.grid(), oracle.count_grid(v)) and np.array_equal(b.grid(), a.grid())
            assert a.info().supersegments == b.info().supersegments == int(v.count.sum())
            assert np.array_equal(render(a, cam, 60, 44), render(b, cam, 60, 44))
            if store == "f32":
                assert np.abs(render(b, cam, 60, 44) - oracle.render_exact(v, cam, 60, 44)).max() <= TOL
            b.replace_begin(d)
            while not b.replace_poll():
                pass
            assert np.array_equal(render(a, cam, 60, 44), render(b, cam, 60, 44))
    bad = d.count.clone()
    bad[0, 0] = 255
    if ns < 255:
        with pytest.raises(V.VdiError) as e:
            V.Vdi(V.DeviceVDI(bad, d.depth, d.rgba, v.camera, v.bmin, v.bmax, v.grid_k, v.grid_nz, v.grid_z))
        assert e.value.code == V.VDI_ERR_ARG


def test_creates_after_destroys():
    """Uploads from host planes after the VDIs, and so the streams, of earlier
    uploads are gone."""
    V = _V()
    v = synth.random_vdi(20, 14, 5, seed=3)
    for _ in range(12):
        with V.Vdi(v) as h:
            assert h.info().supersegments == int(v.count.sum())


@pytest.mark.parametrize("dims", [(1, 9, 7), (2, 5, 11), (3, 1, 1), (17, 2, 33)])
@pytest.mark.parametrize("u16", [False, True])
def test_narrow_volumes(dims, u16):
    V = _V()
    nx, ny, nz = dims
    vol = np.random.default_rng(nx).random((nz, ny, nx)).astype(np.float32)
    vol = (vol * 65535).astype(np.uint16) if u16 else vol
    dvol = torch.from_numpy(vol.view(np.int16) if u16 else vol).cuda()
    bmin, bmax = inputs.aabb_for(dims)
    cam = inputs.orbit_camera(23.0, radius=1.2)
    for tf, name in ((inputs.TF_KNOTS4, "knots4"), (inputs.TF_RAMP, "ramp")):
        for gamma in (0.0, 0.01):
            ref = inputs.generate_vdi(vol, cam, 37, 21, 6, tf, gamma)
            got = V.generate(dvol, bmin, bmax, cam, 37, 21, 6, tf=name, gamma=gamma)
            torch.cuda.synchronize()
            for a, b in zip(got, (ref.count, ref.depth, ref.rgba, ref.gamma)):
                assert np.array_equal(a.cpu().numpy(), b), (tf, gamma)
        f64 = V.dvr(dvol, bmin, bmax, cam, 37, 21, tf=name, precision="f64").cpu().numpy()
        f32 = V.dvr(dvol, bmin, bmax, cam, 37, 21, tf=name, precision="f32").cpu().numpy()
        assert np.array_equal(f64, ref.dvr.astype(np.float32))
        assert np.abs(f32 - ref.dvr).max() <= 1e-4


# Tiles of 32 x 16 pixels, windows of 11 x 11.
@pytest.mark.parametrize("W,H", [(11, 11), (32, 16), (33, 17), (43, 27), (75, 11), (11, 60)])
def test_quality_tiles(W, H):
    rng = np.random.default_rng(W * H)
    a = rng.random((H, W, 4)).astype(np.float32)
    b = np.clip(a + 0.1 * rng.standard_normal(a.shape), 0, 1).astype(np.float32)
    s, p = _V().image_quality(torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda())
    assert s == pytest.approx(Q.ssim(a, b), abs=1e-10) and p == pytest.approx(Q.psnr(a, b), abs=1e-9)
