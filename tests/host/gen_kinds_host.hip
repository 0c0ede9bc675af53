// Host build of the GPU generator's per-ray code as its kernel runs it: the
// instance that vdi_generate launches for the volume and for a device of `lanes`
// lanes, each with a sample cache of the size that it allocates.
#include "vdi_generate.hip"

#include <cstdio>
#include <vector>

namespace vdi {
int set_error(int code, const char *fmt, ...)
{
    fprintf(stderr, "vdi_generate host build: %s\n", fmt);
    return code;
}
int hip_error(hipError_t, const char *) { return VDI_ERR_HIP; }
hipError_t library_pool(int, hipMemPool_t *) { return hipErrorNotSupported; }
}  // namespace vdi

// *entries: the cache's entries a lane; *fits: whether every ray's samples are
// taken to fit it; *over: entries written behind it.
extern "C" int host_generate_kind(const vdi_volume *vol, const vdi_gen_params *p, uint8_t *count, float *depth, float *rgba,
                                  double *gamma_out, uint64_t lanes, int *entries, int *fits, int *over)
{
    vdi::GenParams G;
    const int rc = vdi::make_gen_params(vol, p, G);
    if (rc) return rc;
    const int K = vdi::cache_entries(G, lanes);
    *entries = K;
    *fits = K == G.maxs;
    *over = 0;
    // Behind the cache: room for every sample that a ray may ever have.
    const int room = 2 * std::max(vol->nx, std::max(vol->ny, vol->nz)) + 8;
    std::vector<double2> buf((size_t)K + room);
    const vdi::SampleCache C = {buf.data(), K, 1};
    vdi::by_kind(G, [&](auto kind) {
        constexpr vdi::VoxelKind k = decltype(kind)::value;
        for (int py = 0; py < p->height; ++py)
            for (int px = 0; px < p->width; ++px) {
                for (double2 &e : buf) e = make_double2(-7.0, -7.0);
                auto ray = K == G.maxs ? vdi::gen_ray<true, k> : vdi::gen_ray<false, k>;
                ray(G, G.tab, C, px, py, count, reinterpret_cast<float2 *>(depth), reinterpret_cast<float4 *>(rgba), gamma_out);
                for (size_t i = K; i < buf.size(); ++i) *over += buf[i].x != -7.0;
            }
        return 0;
    });
    return 0;
}
