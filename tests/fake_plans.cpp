// What a launched kernel has been told, for the log of fake_device.cpp (a file of its own: it needs the library's own structures,
// whose header brings the HIP runtime's declarations).
#include <string>

#include "dn_internal.h"

// slice_epoch_kernel: workgroups that take part, and how many of them have units of some hidden layer.  tile_epoch_kernel: whether all the
// workgroups it waits for will come; if not, it says so as it would on a device.
std::string plan_of(const std::string &kernel, void **parameters)
{
    if (kernel == "tile_epoch_kernel") {
        const dn::TilePlan &p = *static_cast<const dn::TilePlan *>(parameters[0]);
        if (p.expected == (unsigned)p.grid) return "all";
        *p.settled = -1;
        *p.abort_flag = 1;
        return "kept-apart";
    }
    if (kernel != "slice_epoch_kernel") return "";
    const dn::SlicePlan &p = *static_cast<const dn::SlicePlan *>(parameters[0]);
    int L = 0, owning = 0;
    while (L < dn::SLICE_MAX_L && p.layer[L + 1].n_out > 0) ++L;
    for (int w = 0; w < p.P; ++w) {
        bool any = false;
        for (int l = 1; l < L; ++l) any = any || w * p.layer[l].per < p.layer[l].n_out;
        owning += any;
    }
    return std::to_string(p.P) + "of" + std::to_string(owning);
}
