// Launch interface of the staged x passes (kernels_xs.hip, kernels_xs2.hip), used by
// the x-pass launchers.
#pragma once

#include "kernels_impl.h"

namespace kw {

// The three x passes of a step (LaunchCfg::xs): the arguments of the x-row
// kernels.  Where a pass runs on planes (LaunchCfg::planes) Sin are spectra before
// the y inverse transform, Sout spectra after the y forward transform (the
// pressure spectrum: x only).  scr: a real field used as scratch (a spectrum
// array that is free at this point).
// points: force sources or a velocity series; mask sensors or pressure sources
hipError_t launch_xs_vel(hipStream_t s, const LaunchCfg &c, const XArgs &a, bool points);
hipError_t launch_xs_den(hipStream_t s, const LaunchCfg &c, const XArgs &a, float *scr);
hipError_t launch_xs_eos(hipStream_t s, const LaunchCfg &c, const XArgs &a, float *scr,
                         bool points, bool merged);
// the same for power-of-two lengths (LaunchCfg::xs == 1)
hipError_t launch_xs2_vel(hipStream_t s, const LaunchCfg &c, const XArgs &a, bool points);
hipError_t launch_xs2_den(hipStream_t s, const LaunchCfg &c, const XArgs &a, float *scr);
hipError_t launch_xs2_eos(hipStream_t s, const LaunchCfg &c, const XArgs &a, float *scr,
                          bool points, bool merged);
// the x passes of a reverse step in LaunchCfg::xs_adj (kernels_xadj.hip)
hipError_t launch_xs_adj(hipStream_t s, int pass, const LaunchCfg &c, const XArgs &a, const AdjDev &ad,
                         const float2 *p_spec, bool loss);

}  // namespace kw
