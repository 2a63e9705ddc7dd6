// collide_fp64.hip -- the FP64 form's batched collision kernel for fixed event
// counts, in a code object of its own: 240 KB of code, which ran the batched
// FP64 workload in 2.72 ms here and in 3.00 to 3.08 (same instructions) beside
// any other kernel.  The mixed form's kernels showed no such difference.
#include "collide_device.hpp"

namespace mcd {

template __global__ void collide_batched<double, 4, false, false, false, kFixedCount>(CollideArgs A);

}  // namespace mcd
