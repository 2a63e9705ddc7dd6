// collide_batched_prob.hip -- the batched collision kernels for the probabilistic fragmentation criteria.
#include "collide_launch.hpp"

namespace mcd {

template <>
hipError_t launch_batched<true>(const CollideArgs &a, int precision, int n_cells, bool wide,
                                 int grid_override, hipStream_t s) {
  return batched_forms<true>(a, precision, n_cells, wide, grid_override, s);
}

}  // namespace mcd
