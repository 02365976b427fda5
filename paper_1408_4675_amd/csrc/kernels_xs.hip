// The staged x passes for the lengths 2^a 3^b 5^c that have stages, and the choice between them and
// the kernels for powers of two (kernels_xs2.hip).
#include "xstaged_impl.h"

namespace kw {

using XAny = XStagedLaunch<kAnyY, kAnyM, kAnyP>;

hipError_t launch_xs_vel(hipStream_t s, const LaunchCfg &c, const XArgs &x, bool points) {
    return c.xs == 1 ? launch_xs2_vel(s, c, x, points) : XAny::vel(s, c, x, points);
}
hipError_t launch_xs_den(hipStream_t s, const LaunchCfg &c, const XArgs &x, float *scr) {
    return c.xs == 1 ? launch_xs2_den(s, c, x, scr) : XAny::den(s, c, x, scr);
}
hipError_t launch_xs_eos(hipStream_t s, const LaunchCfg &c, const XArgs &x, float *scr,
                         bool points, bool merged) {
    return c.xs == 1 ? launch_xs2_eos(s, c, x, scr, points, merged) : XAny::eos(s, c, x, scr, points, merged);
}

}  // namespace kw
