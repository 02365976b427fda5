// Launch interface of the staged z pass (kernels_zs.hip), used by launch_zfused.
#pragma once

#include "kernels_impl.h"

namespace kw {

hipError_t launch_zstaged(hipStream_t s, const LaunchCfg &c, int mode, const ZArgs &z, int n_out);

}  // namespace kw
