// Host build of rays folded on one lane.
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

extern "C" int host_split_launch(double rays, double others) { return vdi::split_launch(rays, others); }
