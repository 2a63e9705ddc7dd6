// collide_ilp.hip -- the mixed form's batched collision kernel for time-limited
// steps without the composition mix and the event log, compiled with the
// scheduling strategy that maximises instruction-level parallelism (the build
// gives this file that flag): it has registers to spare at two waves per SIMD.
#include "collide_device.hpp"

namespace mcd {

template __global__ void collide_batched<float, 4, true, false, false, kTimeLimited>(CollideArgs A);

}  // namespace mcd
