// collide_ilp.hip -- batched collision kernels that are compiled with the
// scheduling strategy that maximises instruction-level parallelism (the build
// gives this file that flag): the mixed form's for time-limited steps without
// the composition mix and the event log, and the FP64 form's for fixed event
// counts.  Both have registers to spare at two waves per SIMD.
#include "collide_device.hpp"

namespace mcd {

template __global__ void collide_batched<float, 4, true, false, false, kTimeLimited>(CollideArgs A);
template __global__ void collide_batched<double, 4, false, false, false, kFixedCount>(CollideArgs A);

}  // namespace mcd
