// drift_pair_f32.hip -- the two-axis position passes of drift_pair.h in FP32, and
// the entry of both types. gfx950.
#include "drift_pair.h"

namespace vp {
namespace {

bool has_length(int n)
{
  return n == 4 || n == 6 || n == 8 || n == 12 || n == 16 || n == 24 || n == 32 || n == 48 || n == 64;
}

}  // namespace

bool drift_pair_supported(int dtype, int na, int nb, long long nv3)
{
  return has_length(na) && has_length(nb) && pair_plane(dtype == 0 ? 4 : 8, na, nb) && nv3 % 256 == 0 &&
         nv3 < (1LL << 31);
}

// wavefronts of the pass over the axes na, nb with o cells on the third
long long drift_pair_waves(int dtype, int na, int nb, int o, long long nv3)
{
  const int w = pair_row(dtype == 0 ? 4 : 8, na * nb);
  return o * (nv3 / 256) * (pair_rows(na < nb ? na : nb, w) * w / 64);
}

// bytes of LDS a workgroup of it holds
int drift_pair_tile(int dtype, int na, int nb)
{
  const int es = dtype == 0 ? 4 : 8;
  return na * nb * pair_row(es, na * nb) * es;
}

hipError_t launch_drift_pair_f32(const DriftPairArgs& p, int na, int nb, hipStream_t s)
{
  return launch_pair_t<float>(p, na, nb, s);
}

hipError_t launch_drift_pair(const DriftPairArgs& p, int dtype, int na, int nb, hipStream_t s)
{
  if (!drift_pair_supported(dtype, na, nb, p.nv3)) return hipErrorInvalidValue;
  return dtype == 0 ? launch_drift_pair_f32(p, na, nb, s) : launch_drift_pair_f64(p, na, nb, s);
}

}  // namespace vp
