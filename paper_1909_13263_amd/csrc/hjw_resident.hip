// hjw_resident.hip - the instantiations of the resident launch's kernels (hjw_resident.h).
// They are a source of their own because they are compiled without the machine-level hoisting
// of loop invariants: out of the loop over stages it moves the FP64 constants and the LDS
// addresses of every sweep and finish, which then live in registers all at once (FP64, 64 x 8 tile:
// 19 VGPRs and 190 SGPRs spilled with it, none and 109 without; 64 x 16: 23 and 278, none and
// 114).
#include "hjw_resident.h"

#include <type_traits>

namespace hjw {
namespace {

template <typename T, typename P, bool OWN>
const void* pick(int dim, int ty, int seg) {
    if (dim == 1) return reinterpret_cast<const void*>(k_resident1d<T, P, OWN>);
    if (ty == 4 && seg == 0) return reinterpret_cast<const void*>(k_resident2d<T, P, 4, 0, OWN>);
    if (ty == 8 && seg == 2) return reinterpret_cast<const void*>(k_resident2d<T, P, 8, 2, OWN>);
    if (ty == 16 && seg == 4) return reinterpret_cast<const void*>(k_resident2d<T, P, 16, 4, OWN>);
    if (ty == 16 && seg == 8) return reinterpret_cast<const void*>(k_resident2d<T, P, 16, 8, OWN>);
    return nullptr;
}
template <typename T, typename P>
const void* pick(int dim, int ty, int seg, bool own) {
    return own ? pick<T, P, true>(dim, ty, seg) : pick<T, P, false>(dim, ty, seg);
}

}  // namespace

const void* resident_kernel(int prec, int dim, int ty, int seg, bool own) {
    switch (prec) {
    case HJW_FP64:
        return pick<double, double>(dim, ty, seg, own);
    case HJW_FP32_MIXED:
        return pick<float, double>(dim, ty, seg, own);
    default:
        return pick<float, float>(dim, ty, seg, own);
    }
}

}  // namespace hjw
