// Host build of the ray walkers' arithmetic of bounds: the floats next to a
// depth.
#include "vdi_trace.h"

extern "C" void host_float_bounds(const double *z, int n, float *below, float *above)
{
    for (int i = 0; i < n; ++i) {
        below[i] = vdi::float_below(z[i]);
        above[i] = vdi::float_above(z[i]);
    }
}
