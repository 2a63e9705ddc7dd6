// collide_batched.hip -- the batched collision kernels for the sharp fragmentation criterion.
#include "collide_launch.hpp"

namespace mcd {

template <>
hipError_t launch_batched<false>(const CollideArgs &a, int precision, int n_cells, bool wide,
                                 int grid_override, hipStream_t s) {
  return batched_forms<false>(a, precision, n_cells, wide, grid_override, s);
}

}  // namespace mcd
