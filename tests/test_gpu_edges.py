"""Calls at the edges of what the entry points accept (needs an MI355X): eyes
far from the volume; device planes that are not memory of the device or not
aligned to a slot, or are still being written on the null stream; volumes with
infinite and NaN voxels; so many small exact frames at once that their rays'
parts are folded on one lane; a VDI too large for 32-bit offsets; sensitivities at Eq. 1's
own distances."""
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


def dvr_f32_reference(vol, bmin, bmax, cam, W, H, tf):
    """FP32 DVR in numpy: rays and sample positions in float64, interpolation lo (1 - w) + hi w, transfer function,
    opacity and compositing in float32."""
    f4 = np.float32
    e, t, u = (np.array(x, dtype=np.float64) for x in (cam.eye, cam.target, cam.up))
    F = (t - e) / np.linalg.norm(t - e)
    R = np.cross(F, u)
    R /= np.linalg.norm(R)
    U = np.cross(R, F)
    th = np.tan(float(f4(cam.fov_y_deg)) * np.pi / 360)
    xc, yc = -1 + (2 * np.arange(W) + 1) / W, -1 + (2 * np.arange(H) + 1) / H
    d = F + xc[None, :, None] * th * W / H * R + yc[:, None, None] * th * U
    d /= np.linalg.norm(d, axis=2, keepdims=True)
    lo, hi = float(f4(cam.near)) / (d @ F), np.full((H, W), np.inf)
    for a in range(3):
        ta, tb = (bmin[a] - e[a]) / d[..., a], (bmax[a] - e[a]) / d[..., a]
        lo, hi = np.maximum(lo, np.minimum(ta, tb)), np.minimum(hi, np.maximum(ta, tb))
    hit = hi > lo
    n = np.array(vol.shape[::-1])
    ds = max(b - a for a, b in zip(bmin, bmax)) / n.max()
    N = np.where(hit, np.maximum(np.ceil((hi - lo) / ds - 1e-9), 1), 0)
    with np.errstate(all="ignore"):
        ln = np.where(hit, (hi - lo) / N, 0)
        r = (ln / ds).astype(f4)
        acc, T = np.zeros((H, W, 3), f4), np.ones((H, W), f4)
        sc = n / (np.array(bmax) - np.array(bmin))
        u0 = (e + (np.where(hit, lo, 0) + 0.5 * ln)[..., None] * d - np.array(bmin)) * sc - 0.5
        du = ln[..., None] * d * sc
        for q in range(int(N.max())):
            live = (q < N) & (T > f4(1e-5))
            uv = u0 + q * du
            i0 = np.floor(uv).astype(int)
            w = (uv - i0).astype(f4)
            a, b = np.clip(i0, 0, n - 1), np.clip(i0 + 1, 0, n - 1)
            at = lambda x, y, z: vol[z[..., 2], y[..., 1], x[..., 0]]
            mix = lambda p, q_, k: p * (1 - w[..., k]) + q_ * w[..., k]
            c = [mix(at(a, y, z), at(b, y, z), 0) for z in (a, b) for y in (a, b)]
            v = mix(mix(c[0], c[1], 1), mix(c[2], c[3], 1), 2)
            if tf == "ramp":
                col = np.stack((v, f4(0.25) + f4(0.5) * v, 1 - v), -1)
                op = f4(0.2) * np.fmin(np.fmax((v - f4(0.05)) / f4(0.95), f4(0)), f4(1))
            else:
                v = np.fmin(np.fmax(v, f4(0)), f4(1))
                kv, ka = np.array([0, 0.25, 0.55, 1], f4), np.array([0, 0, 0.04, 0.12], f4)
                kc = np.array([[0.1, 0.2, 0.8], [0.1, 0.7, 0.9], [0.95, 0.9, 0.3], [0.9, 0.15, 0.1]], f4)
                s = (v >= kv[1]).astype(int) + (v >= kv[2])
                x = (v - kv[s]) / (kv[s + 1] - kv[s])
                col, op = kc[s] + x[..., None] * (kc[s + 1] - kc[s]), ka[s] + x * (ka[s + 1] - ka[s])
            al = np.where(op > 0, 1 - np.power(1 - op, r), f4(0)).astype(f4)
            acc = np.where(live[..., None], acc + (T * al)[..., None] * col, acc)
            T = np.where(live, T * (1 - al), T)
    return np.concatenate((acc, (1 - T)[..., None]), 2)


# Infinite and NaN voxels, and neighbours whose difference overflows FP32.
@pytest.mark.parametrize("tf,values", [("knots4", (np.inf, -np.inf)), ("knots4", (np.inf,)), ("knots4", (np.nan,)),
                                       ("knots4", (3e38, -3e38)), ("ramp", (np.inf,)), ("ramp", (-np.inf,)),
                                       ("ramp", (np.nan,))])
@pytest.mark.parametrize("dims", [(12, 11, 10), (1, 11, 10)])
def test_dvr_of_volumes_with_values_out_of_range(dims, tf, values):
    V = _V()
    nx, ny, nz = dims
    rng = np.random.default_rng(17)
    vol = (0.5 + 0.3 * rng.random((nz, ny, nx))).astype(np.float32)
    for k in range(6):
        vol[tuple(rng.integers(0, n) for n in vol.shape)] = values[k % len(values)]
    bmin, bmax = inputs.aabb_for(dims)
    cam = inputs.orbit_camera(23.0, radius=1.6)
    generated = inputs.generate_vdi(vol, cam, 61, 47, 6, inputs.TF_RAMP if tf == "ramp" else inputs.TF_KNOTS4, 0.01)
    for precision, ref in (("f64", generated.dvr.astype(np.float32)),
                           ("f32", dvr_f32_reference(vol, bmin, bmax, cam, 61, 47, tf))):
        got = V.dvr(on_device(vol), bmin, bmax, cam, 61, 47, tf=tf, precision=precision).cpu().numpy()
        same = {k: bool(np.array_equal(f(got), f(ref))) for k, f in (("nan", np.isnan), ("inf", np.isposinf), ("-inf", np.isneginf))}
        fin = np.isfinite(ref) & np.isfinite(got)
        off = float(np.abs(got[fin] - ref[fin]).max())
        print(f"[gpu] {precision} {tf} {values} {dims}: {same}, {int((~np.isfinite(ref)).sum())} not finite, off {off:.1e}",
              flush=True)
        assert fin.any() and all(same.values()) and off <= 1e-4, precision


# 70 frames of 128 x 128 and 8 of 97 x 55 to 300 x 216: more rays in parts than a launch splits.
@pytest.mark.parametrize("store", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("alpha_max", [0.12, 0.95])
def test_many_small_frames_are_their_single_renders(store, alpha_max):
    V = _V()
    from paper_2206_08660_amd import serve as S
    v = synth.random_vdi(131, 97, 24, seed=84, alpha_max=alpha_max, empty_frac=0.3)
    frames = [(inputs.orbit_camera(-44.0 + 1.2 * i), 128, 128, 1.0, 0.0) for i in range(70)]
    frames += [(inputs.orbit_camera(7.0 * i - 20.0), 97 + 29 * i, 55 + 23 * i, 1.0, 0.0) for i in range(8)]
    frames += [(inputs.orbit_camera(11.0), 640, 480, 1.0, 0.0), (inputs.orbit_camera(12.0), 256, 256, 2.0, 0.0),
               (inputs.orbit_camera(-9.0), 200, 150, 1.0, 2.0), (inputs.orbit_camera(31.0), 320, 200, 2.0, 1.0)]
    with V.Vdi(v, store=store) as h:
        want = [h.render(cam, w, hh, d_i=di, d_r=dr) for cam, w, hh, di, dr in frames]

        def outs():
            return [torch.full((f[2], f[1], 4), -1.0, device="cuda") for f in frames]
        for n in (len(frames), 20):     # the first 20 are few enough to be split
            got = outs()
            V.render_batch([(h, cam, w, hh, di, dr, o) for (cam, w, hh, di, dr), o in zip(frames[:n], got)])
            torch.cuda.synchronize()
            assert all(torch.equal(a, b) for a, b in zip(got[:n], want[:n]))
        for persistent in (False, True):
            print(f"[gpu] server, persistent {persistent}, {store}, alpha {alpha_max}", flush=True)
            got = outs()
            with S.Server(4 << 30, max_inflight=96, persistent=persistent) as s:
                for (cam, w, hh, di, dr), o in zip(frames, got):
                    assert s.submit(h, cam, w, hh, di, dr, o) is not None
                s.drain()
            torch.cuda.synchronize()
            assert all(torch.equal(a, b) for a, b in zip(got, want))


@pytest.mark.parametrize("store", ["f32", "f16", "bf16"])
def test_a_vdi_too_large_for_32_bit_offsets(store):
    """The same lists with N_S 20 and with N_S 255 (over 2^28 slots, which the kernels address in 64 bits), bit for
    bit: single and batched frames, whole, split and folded rays, previews."""
    V = _V()
    tile = synth.random_vdi(161, 104, 20, seed=85, alpha_max=0.2, empty_frac=0.2)
    count, depth, rgba = (np.tile(a, (8, 8) if a.ndim == 2 else (1, 8, 8, 1)) for a in (tile.count, tile.depth, tile.rgba))
    small = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (count, depth, rgba)]
    big = [small[0]] + [torch.zeros((255, *t.shape[1:]), device="cuda") for t in small[1:]]
    for b, t in zip(big[1:], small[1:]):
        b[:20] = t
    rest = (tile.camera, tile.bmin, tile.bmax, tile.grid_k, tile.grid_nz, tile.grid_z)
    exact = [(inputs.orbit_camera(a), w, hh, 1.0, 0.0) for a, w, hh in ((8.0, 128, 128), (31.0, 900, 600), (-20.0, 60, 41))]
    previews = [(inputs.orbit_camera(a), 800, 450, di, dr) for a, di, dr in ((8.0, 1.0, 1.0), (-31.0, 2.0, 2.0))]
    many = [(inputs.orbit_camera(0.5 * i), 128, 128, 1.0, 0.0) for i in range(30)]
    images = []
    for planes in (small, big):
        with V.Vdi(V.DeviceVDI(*planes, *rest), store=store) as h:
            got = [h.render(f[0], f[1], f[2], d_i=f[3], d_r=f[4]) for f in exact + previews + many]
            got.append(h.render(*exact[1][:3], ess=False))
            got.append(h.render(*exact[0][:3], ess=False))
            for frames in (exact[:1], exact[1:2], exact + previews, previews, many):
                outs = [torch.full((f[2], f[1], 4), -1.0, device="cuda") for f in frames]
                V.render_batch([(h, *f, o) for f, o in zip(frames, outs)])
                got += outs
            torch.cuda.synchronize()
            print(f"[gpu] {store}, N_S {h.ns}: {len(got)} images", flush=True)
        images.append([g.cpu() for g in got])
    assert all(torch.equal(a, b) for a, b in zip(*images))
    singles = dict(zip(map(id, exact + previews + many), images[1]))
    batched = images[1][len(singles) + 2:]
    for f, b in zip(exact[:1] + exact[1:2] + exact + previews + previews + many, batched):
        assert torch.equal(singles[id(f)], b)


@pytest.mark.parametrize("tf,name", [(inputs.TF_KNOTS4, "knots4"), (inputs.TF_RAMP, "ramp")])
def test_sensitivities_at_the_distances_themselves(tf, name):
    """Eq. 1 is decided in FP32 only beyond a bound on its error.  gamma is set to distances of the generator (found
    by bisection, to neighbouring doubles) and to both sides of them, up to where the bound ends."""
    V = _V()
    rng = np.random.default_rng(21)
    vol = (0.2 + 0.6 * rng.random((32, 32, 32))).astype(np.float32)
    bmin, bmax = inputs.aabb_for((32, 32, 32))
    dvol = on_device(vol)
    cam = inputs.orbit_camera(31.0)
    W, H, ns = 12, 9, 30

    def counts(gamma):
        return inputs.generate_vdi(vol, cam, W, H, ns, tf, gamma)

    gammas = []
    pixels = np.argwhere(counts(1e-4).count > 4)
    for y, x in pixels[rng.permutation(len(pixels))[:12]]:
        lo, hi = 10.0 ** rng.uniform(-4, -1.5), 1.0
        n = counts(lo).count[y, x]
        if n == 1:
            continue
        while np.nextafter(lo, hi) < hi:
            g = 0.5 * (lo + hi)
            if counts(g).count[y, x] == n:
                lo = g
            else:
                hi = g
        gammas += [lo, hi] + [hi + s * e for e in (1e-9, 5e-8, 2e-7, 1e-6, 3.4e-6, 3.6e-6) for s in (-1, 1)]
    assert len(gammas) > 60
    for g in gammas:
        if g <= 0.0:
            continue
        ref = counts(g)
        got = V.generate(dvol, bmin, bmax, cam, W, H, ns, tf=name, gamma=g)
        torch.cuda.synchronize()
        for a, b in zip(got, (ref.count, ref.depth, ref.rgba, ref.gamma)):
            assert np.array_equal(a.cpu().numpy(), b), g
    print(f"[gpu] {name}: {len(gammas)} sensitivities", flush=True)
