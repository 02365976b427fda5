// Launch interface of the staged y pass (kernels_ys.hip), used by launch_ypass.
#pragma once

#include "kernels_impl.h"

namespace kw {

hipError_t launch_ystaged(hipStream_t s, const LaunchCfg &c, const YArgs &y, bool inverse, int nfields);

}  // namespace kw
