// collide_ilp3.hip -- the mixed form's batched collision kernels that run three
// waves per SIMD: for fixed event counts, and for time-limited steps with the
// composition mix.  As collide_ilp.hip, and with constants formed where they
// are used instead of being held (and spilled) through the events: 0 and 28
// bytes of spill per lane instead of 92 and 112.  A kernel's spill is also
// device memory, reserved for every wave the GPU can hold.
#include "collide_device.hpp"

namespace mcd {

template __global__ void collide_batched<float, 4, true, false, true, kTimeLimited>(CollideArgs A);
template __global__ void collide_batched<float, 4, true, false, false, kFixedCount>(CollideArgs A);

}  // namespace mcd
