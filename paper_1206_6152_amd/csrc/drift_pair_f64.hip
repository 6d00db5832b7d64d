// drift_pair_f64.hip -- the two-axis position passes of drift_pair.h in FP64. gfx950.
#include "drift_pair.h"

namespace vp {

hipError_t launch_drift_pair_f64(const DriftPairArgs& p, int na, int nb, hipStream_t s)
{
  return launch_pair_t<double>(p, na, nb, s);
}

}  // namespace vp
