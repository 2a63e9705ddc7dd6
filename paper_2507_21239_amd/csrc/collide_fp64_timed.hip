// collide_fp64_timed.hip -- the FP64 form's batched collision kernel for
// time-limited steps.  Its instructions are left where the compiler places them:
// 140 bytes of spill a lane, but a lone cell's events 2% faster than with
// instructions sunk into the loop (one cell of 200, constant kernel: 5835 against
// 5941 us; a disk of 1e5: 4.26 against 4.32 ms).
#include "collide_device.hpp"

namespace mcd {

template __global__ void collide_batched<double, 4, false, false, false, kEitherLimit>(CollideArgs A);

}  // namespace mcd
