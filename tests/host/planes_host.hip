// Host build of the rule on which planes of a VDI an upload's kernels read in
// place.
#include "vdi_internal.h"

extern "C" int host_in_place(int type, int managed, int plane_device, uint64_t address, int device, uint64_t align)
{
    hipPointerAttribute_t a = {};
    a.type = (hipMemoryType)type;
    a.isManaged = managed;
    a.device = plane_device;
    return vdi::readable_in_place(a, reinterpret_cast<const void *>(address), device, align);
}
