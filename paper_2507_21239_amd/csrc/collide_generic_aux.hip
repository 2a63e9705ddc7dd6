// collide_generic_aux.hip -- the mixed form's batched collision kernels with the
// composition mix or the event log for the test kernels and partial velocity
// sources, both kinds of fragmentation criterion.  Their instructions are left
// where the compiler places them: sunk into the loops, those of the row sums' pairs
// are repeated for every partner (row sums of 200 cells of 263 - 1024 particles
// 928 against 1003 us, 100 events with them 1299 against 1425).
#include "collide_device.hpp"

namespace mcd {

template __global__ void collide_batched<float, 4, false, false, true, kEitherLimit>(CollideArgs A);
template __global__ void collide_batched<float, 4, false, true, true, kEitherLimit>(CollideArgs A);

}  // namespace mcd
