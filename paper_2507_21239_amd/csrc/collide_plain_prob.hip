// collide_plain_prob.hip -- the one-workgroup-per-cell collision kernels, probabilistic criteria.
#include "collide_launch.hpp"

namespace mcd {

template <>
hipError_t launch_plain<true>(const CollideArgs &a, int precision, int n_cells, bool wide,
                               hipStream_t s) {
  return plain_forms<true>(a, precision, n_cells, wide, s);
}

}  // namespace mcd
