// Instances of the resident-score kernel: one object per caller (RR_MODE), input
// type (RR_DT) and representation width (RR_D), set by the build.
#include "rr_resident_impl.hpp"

#define RR_CAT5(a, b, c, d, e) a##b##_##c##_##d
#define RR_NAME(mode, dt, d) RR_CAT5(launch_resident_, mode, dt, d, )

namespace rr {

hipError_t RR_NAME(RR_MODE, RR_DT, RR_D)(const RouteArgs &a, hipStream_t stream)
{
    return resident::launch_d<RR_MODE, RR_DT, RR_D>(a, stream);
}

}  // namespace rr
