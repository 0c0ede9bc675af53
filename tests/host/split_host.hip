// Host build of what decides how an exact frame is dealt out: split rays with
// 32- and 64-bit plane offsets, the order of a frame's tiles, and the bounds of
// the AABB on the image.
#include "vdi_kernels.hip"
#include "vdi_api.hip"

#include <vector>

namespace {

struct HostVdi {
    vdi::VdiSet v;
    std::vector<float2> dep;
    std::vector<float4> col;
    std::vector<uint32_t> bits;
};

int load(const vdi_desc *d, const uint32_t *grid, HostVdi &h)
{
    h.v.cam_o = d->camera_VO;
    memcpy(h.v.bmin, d->aabb_min, sizeof h.v.bmin);
    memcpy(h.v.bmax, d->aabb_max, sizeof h.v.bmax);
    vdi::DevVDI &D = h.v.dev;
    D.WO = d->width;
    D.HO = d->height;
    D.NS = d->max_supersegments;
    D.fmt = VDI_F32;
    D.plane = (uint64_t)d->width * d->height;
    D.sstride = vdi::kBrick;
    const uint64_t elems = vdi::plane_elems(D.WO, D.HO, D.NS);
    h.dep.assign(elems, make_float2(NAN, NAN));
    h.col.assign(elems, make_float4(NAN, NAN, NAN, NAN));
    for (int j = 0; j < D.NS; ++j)
        for (uint64_t li = 0; li < D.plane; ++li) {
            const uint64_t o = vdi::list_base(li, D.NS, D.WO) + (uint64_t)j * D.sstride;
            h.dep[o] = reinterpret_cast<const float2 *>(d->depth)[(uint64_t)j * D.plane + li];
            h.col[o] = static_cast<const float4 *>(d->rgba)[(uint64_t)j * D.plane + li];
        }
    D.gk = d->grid_k;
    D.gnz = d->grid_nz;
    D.GW = (d->width + d->grid_k - 1) / d->grid_k;
    D.GH = (d->height + d->grid_k - 1) / d->grid_k;
    const uint32_t ncells = (uint32_t)(D.gnz * D.GH * D.GW);
    h.bits.assign((ncells + 31) / 32, 0u);
    for (uint32_t c = 0; c < ncells; ++c)
        if (grid[c] != 0u) h.bits[c / 32] |= 1u << (c % 32);
    D.count = d->count;
    D.depth = h.dep.data();
    D.rgba = h.col.data();
    D.grid = grid;
    D.gbits = h.bits.data();
    D.gz = d->grid_z;
    Basis ob;
    const int rc = make_basis(d->camera_VO, ob);
    if (rc) return rc;
    D.tx_o = (float)(ob.th * ((double)d->width / d->height));
    D.ty_o = (float)ob.th;
    D.dcx = 2.0 / d->width;
    D.dcy = 2.0 / d->height;
    D.inv_gk = nextafterf(1.0f / (float)d->grid_k, INFINITY);
    return VDI_OK;
}

// A ray in `parts` parts, combined as split_tile does.
template <typename Idx>
vdi::Accum split_ray(const vdi::DevVDI &D, const vdi::Frame &f, const float *gz, int px, int py, int parts)
{
    vdi::Accum pre = {0.0f, 0.0f, 0.0f, 1.0f};
    for (int k = 0; k < parts; ++k) {
        vdi::Counters cnt = {0, 0};
        vdi::Accum a = {0.0f, 0.0f, 0.0f, 1.0f};
        vdi::trace_exact_part<VDI_F32, VDI_SEARCH_WINDOW, true, false, Idx>(D, f, gz, px, py, k, parts, a, cnt);
        if (k > 0 && pre.T > vdi::kTTerm && pre.T * a.T <= vdi::kTTerm) {
            a = pre;
            vdi::trace_exact_part<VDI_F32, VDI_SEARCH_WINDOW, true, false, Idx>(D, f, gz, px, py, k, parts, a, cnt);
            return a;
        }
        vdi::append(pre, a);
    }
    return pre;
}

}  // namespace

extern "C" int host_split(const vdi_desc *d, const uint32_t *grid, const vdi_camera *cam, int W, int H, int parts, int wide,
                          float *out, int *parts_chosen)
{
    HostVdi h;
    int rc = load(d, grid, h);
    if (rc) return rc;
    vdi::Frame f;
    rc = build_frame(h.v, *cam, W, H, (double)W / H, f);
    if (rc) return rc;
    *parts_chosen = f.xparts;
    for (int py = 0; py < H; ++py)
        for (int px = 0; px < W; ++px) {
            const float4 o = vdi::to_rgba(wide ? split_ray<uint64_t>(h.v.dev, f, d->grid_z, px, py, parts)
                                               : split_ray<uint32_t>(h.v.dev, f, d->grid_z, px, py, parts));
            memcpy(out + 4 * ((size_t)py * W + px), &o, sizeof o);
        }
    return 0;
}

// Tiles of a W x H frame with AABB bounds r[4] = x0, y0, x1, y1: how often each
// tile is placed, and 1 more than 100 times that if it was said to miss.
extern "C" void host_tiles(int W, int H, const int *r, int tw, int th, int band, int *placed)
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
        const bool meets = vdi::place_tile(f, tw, th, band, i, x0, y0);
        if (x0 < 0 || y0 < 0 || x0 >= W || y0 >= H || x0 % tw || y0 % th) continue;
        placed[(y0 / th) * nx + x0 / tw] += meets ? 100 : 101;
    }
}

// Rays of a frame that meet the AABB at pixels outside its bounds.
extern "C" int host_bounds(const vdi_desc *d, const uint32_t *grid, const vdi_camera *cam, int W, int H, int *inside)
{
    HostVdi h;
    vdi::Frame f;
    if (load(d, grid, h) || build_frame(h.v, *cam, W, H, (double)W / H, f)) return -1;
    int lost = 0;
    *inside = std::max(f.rx1 - f.rx0, 0) * std::max(f.ry1 - f.ry0, 0);
    for (int py = 0; py < H; ++py)
        for (int px = 0; px < W; ++px) {
            vdi::Ray r;
            const bool hit = vdi::ray_setup(f, vdi::pixel_ndc(px, W, f.inv_w), vdi::pixel_ndc(py, H, f.inv_h), r);
            lost += hit && !(px >= f.rx0 && px < f.rx1 && py >= f.ry0 && py < f.ry1);
        }
    return lost;
}
