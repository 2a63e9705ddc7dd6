// collide.hip -- choice of the collision kernel (collide_device.hpp) for a
// launch: the batched persistent launch or one workgroup per cell, and the
// test path that writes one cell's full rate matrix.  The kernels are
// instantiated in files of their own (collide_launch.hpp), those of the mixed
// form's common path in collide_ilp.hip and collide_ilp3.hip.
#include <algorithm>

#include "collide_launch.hpp"

namespace mcd {

__global__ void reset_queues(DevState *st) {
  st->big_head = 0;
  st->small_head = 0;
}

// ---------------------------------------------------------------------------
// test path: the full rate matrix of one cell, from the same records and
// pair code as the collision kernel
// ---------------------------------------------------------------------------
template <typename RT, bool FAST>
__global__ __launch_bounds__(256) void rates_cell(CollideArgs A, int cell, double *r_out,
                                                  int64_t ld, double *rowsum) {
  if (A.plan->bad) return;
  const int s0 = A.cell_start[cell];
  const int n = A.cell_start[cell + 1] - s0;
  Gas g;
  gas_from_primaries(A.P, A.gas + (size_t)cell * 6, g);
  const PairConst<RT> pc = make_pair_const<RT>(A.P, g);
  double scale = 1.0;
  if (sizeof(RT) == 4) {
    double ndmax = 0.0;
    for (int k = 0; k < n; ++k) {
      const int p = A.order[s0 + k];
      ndmax = fmax(ndmax, A.M[p] / (A.m[p] * g.V));
    }
    int e2 = 0;
    frexp(ndmax, &e2);
    scale = ldexp(1.0, -e2);
  }
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    const int pi = A.order[s0 + i];
    const Rec<RT> ri = make_rec<RT>(A.P, g, A.m[pi], A.M[pi], scale);
    RT acc = (RT)0;
    for (int k = 0; k < n; ++k) {
      const int pk = A.order[s0 + k];
      const Rec<RT> rk = make_rec<RT>(A.P, g, A.m[pk], A.M[pk], scale);
      RT dv, x, y;
      PairEval<RT, FAST>::run(pc, ri, rk, dv, x, y);
      acc += x;
      r_out[(int64_t)i * ld + k] = (double)x / scale;
    }
    if (rowsum) rowsum[i] = (double)acc / scale;
  }
}

hipError_t launch_collide(const CollideArgs &a, int precision, int schedule, int n_cells,
                          int max_cell, int grid_override, hipStream_t s, bool queues_clear) {
  // slots per lane: four-wave teams hold big_cap particles, single waves
  // small_cap; kernels exist for up to 4 and up to 8
  const int k_big = (a.big_cap + 255) / 256, k_small = (a.small_cap + 63) / 64;
  const int kneed = schedule == 0 ? std::max(k_big, (max_cell + 255) / 256) : std::max(k_big, k_small);
  if (kneed > 8) return hipErrorInvalidValue;
  const bool wide = kneed > 4;
  // the probabilistic fragmentation criteria apply only to the physical kernel
  const bool prob = a.P.frag_mode != FRAG_SHARP && a.P.kernel == K_PHYSICAL;
  if (schedule == 0)
    return prob ? launch_plain<true>(a, precision, n_cells, wide, s)
                : launch_plain<false>(a, precision, n_cells, wide, s);
  if (!queues_clear) {
    reset_queues<<<1, 1, 0, s>>>(a.state);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return prob ? launch_batched<true>(a, precision, n_cells, wide, grid_override, s)
              : launch_batched<false>(a, precision, n_cells, wide, grid_override, s);
}

hipError_t launch_rates_cell(const CollideArgs &a, int precision, int cell, double *r_out,
                             int64_t ld, double *rowsum_out, hipStream_t s) {
  if (precision == 0)
    rates_cell<double, false><<<1, 256, 0, s>>>(a, cell, r_out, ld, rowsum_out);
  else if (fast_path(a, precision))
    rates_cell<float, true><<<1, 256, 0, s>>>(a, cell, r_out, ld, rowsum_out);
  else
    rates_cell<float, false><<<1, 256, 0, s>>>(a, cell, r_out, ld, rowsum_out);
  return hipGetLastError();
}

}  // namespace mcd
