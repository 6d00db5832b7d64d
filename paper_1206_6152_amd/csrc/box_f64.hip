// box_f64.hip -- the run-time-shaped passes of box.h for FP64-stored f.
#include "box.h"

namespace vp {

hipError_t launch_kick_box_f64(const KickArgs& a, const int nv[3], hipStream_t s);
hipError_t launch_drift_box_f64(const DriftBoxArgs& a, int w, hipStream_t s);

hipError_t launch_kick_box_f64(const KickArgs& a, const int nv[3], hipStream_t s)
{
  return launch_kick_box_t<double>(a, nv, s);
}

hipError_t launch_drift_box_f64(const DriftBoxArgs& a, int w, hipStream_t s)
{
  return launch_drift_box_t<double>(a, w, s);
}

}  // namespace vp
