// Host build of rays folded on one lane, of the order of a frame's tiles and of
// 32-bit plane offsets.
#include "split_host.hip"

// The exact frame with its rays in `parts` parts: folded into `folded`, and part
// by part as split_tile combines them into `split`.
extern "C" int host_fold(const vdi_desc *d, const uint32_t *grid, const vdi_camera *cam, int W, int H, int parts, int ess,
                         float *folded, float *split)
{
    HostVdi h;
    vdi::Frame f;
    if (load(d, grid, h) || build_frame(h.v, *cam, W, H, (double)W / H, f)) return -1;
    for (int py = 0; py < H; ++py)
        for (int px = 0; px < W; ++px) {
            vdi::Accum a = {0.0f, 0.0f, 0.0f, 1.0f};
            vdi::Counters cnt = {0, 0};
            if (ess)
                vdi::trace_exact_part<VDI_F32, VDI_SEARCH_WINDOW, true, false, uint32_t, true>(h.v.dev, f, d->grid_z, px, py, 0,
                                                                                               parts, a, cnt);
            else
                vdi::trace_exact_part<VDI_F32, VDI_SEARCH_WINDOW, false, false, uint32_t, true>(h.v.dev, f, d->grid_z, px, py, 0,
                                                                                                parts, a, cnt);
            const float4 o = vdi::to_rgba(a), s = vdi::to_rgba(split_ray<uint32_t>(h.v.dev, f, d->grid_z, px, py, parts));
            memcpy(folded + 4 * ((size_t)py * W + px), &o, sizeof o);
            memcpy(split + 4 * ((size_t)py * W + px), &s, sizeof s);
        }
    return 0;
}

// host_tiles with the order as an argument: as previews', split frames' or exact frames' tiles.
extern "C" void host_tiles_order(int W, int H, const int *r, int tw, int th, int band, int order, int *placed)
{
    vdi::Frame f = {};
    f.W = W;
    f.H = H;
    f.rx0 = r[0];
    f.ry0 = r[1];
    f.rx1 = r[2];
    f.ry1 = r[3];
    const int nx = (W + tw - 1) / tw, n = nx * ((H + th - 1) / th);
    for (int i = 0; i < n; ++i) {
        int x0 = -1, y0 = -1;
        const bool meets = vdi::place_tile(f, tw, th, band, i, x0, y0, order == 1, order == 2);
        if (x0 < 0 || y0 < 0 || x0 >= W || y0 >= H || x0 % tw || y0 % th) continue;
        placed[(y0 / th) * nx + x0 / tw] += meets ? 100 : 101;
    }
}

// Whether a VDI of these sizes is rendered with 32-bit offsets; the largest
// element offset of a slot in 32 and in 64 bits, and the plane's elements.
extern "C" int host_fits32(int WO, int HO, int NS, uint64_t *o)
{
    o[0] = o[1] = 0;
    for (int iy = HO > 2 ? HO - 2 : 0; iy < HO; ++iy)
        for (int ix = WO > 2 ? WO - 2 : 0; ix < WO; ++ix) {
            const uint32_t a = vdi::list_base_xy<uint32_t>(ix, iy, NS, WO) + (uint32_t)(NS - 1) * vdi::kBrick;
            const uint64_t b = vdi::list_base_xy<uint64_t>(ix, iy, NS, WO) + (uint64_t)(NS - 1) * vdi::kBrick;
            o[0] = std::max<uint64_t>(o[0], a);
            o[1] = std::max(o[1], b);
        }
    o[2] = vdi::plane_elems(WO, HO, NS);
    return vdi::fits32(WO, HO, NS);
}

extern "C" int host_split_launch(double rays, double others) { return vdi::split_launch(rays, others); }

// The lists that a frame's rays cross as its set-up estimates them, and by the
// rays themselves.
extern "C" int host_lists(const vdi_desc *d, const uint32_t *grid, const vdi_camera *cam, int W, int H, double *estimate,
                          double *rays)
{
    HostVdi h;
    vdi::Frame f;
    if (load(d, grid, h) || build_frame(h.v, *cam, W, H, (double)W / H, f)) return -1;
    *estimate = f.lists;
    *rays = 0.0;
    for (int i = 0; i < 9; ++i) {
        const double px = f.rx0 + (f.rx1 - f.rx0) * (0.1 + 0.4 * (i % 3)), py = f.ry0 + (f.ry1 - f.ry0) * (0.1 + 0.4 * (i / 3));
        vdi::Ray r;
        if (!vdi::ray_setup(f, -1.0 + 2.0 * px / W, -1.0 + 2.0 * py / H, r)) continue;
        const double z0 = f.Z0 + r.t0 * r.Zp, z1 = f.Z0 + r.t1 * r.Zp;
        *rays = std::max(*rays, fabs((f.X0 + r.t1 * r.Xp) / z1 - (f.X0 + r.t0 * r.Xp) / z0) * d->width / 2 +
                                    fabs((f.Y0 + r.t1 * r.Yp) / z1 - (f.Y0 + r.t0 * r.Yp) / z0) * d->height / 2);
    }
    return 0;
}
