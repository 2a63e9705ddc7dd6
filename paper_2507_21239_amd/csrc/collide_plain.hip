// collide_plain.hip -- the one-workgroup-per-cell collision kernels, sharp criterion.
#include "collide_launch.hpp"

namespace mcd {

template <>
hipError_t launch_plain<false>(const CollideArgs &a, int precision, int n_cells, bool wide,
                               hipStream_t s) {
  return plain_forms<false>(a, precision, n_cells, wide, s);
}

}  // namespace mcd
