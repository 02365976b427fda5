// The staged x passes for power-of-two lengths: fewer radices, fewer registers (a
// radix that is never run still counts, see EngFixed).
#include "xstaged_impl.h"

namespace kw {

using X2 = XStagedLaunch<kPow2Y, kPow2M, kPow2P>;

hipError_t launch_xs2_vel(hipStream_t s, const LaunchCfg &c, const XArgs &x, bool points) {
    return X2::vel(s, c, x, points);
}
hipError_t launch_xs2_den(hipStream_t s, const LaunchCfg &c, const XArgs &x, float *scr) {
    return X2::den(s, c, x, scr);
}
hipError_t launch_xs2_eos(hipStream_t s, const LaunchCfg &c, const XArgs &x, float *scr,
                          bool points, bool merged) {
    return X2::eos(s, c, x, scr, points, merged);
}

}  // namespace kw
