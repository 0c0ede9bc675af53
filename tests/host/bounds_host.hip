// Host build of the ray walkers' arithmetic of bounds: the floats next to a
// depth, and the clipping of a ray's parameter range.
#include "vdi_trace.h"

extern "C" void host_float_bounds(const double *z, int n, float *below, float *above)
{
    for (int i = 0; i < n; ++i) {
        below[i] = vdi::float_below(z[i]);
        above[i] = vdi::float_above(z[i]);
    }
}

extern "C" void host_clip(const double *a, const double *b, int n, double *lo, double *hi, int *ok)
{
    for (int i = 0; i < n; ++i) ok[i] = vdi::clip(a[i], b[i], lo[i], hi[i]);
}
