// collide_launch.hpp -- launches of the collision kernels' instantiations;
// each instantiating file takes one schedule and one kind of fragmentation
// criterion, so that the files build side by side.
#pragma once
#include <algorithm>

#include "collide_device.hpp"

namespace mcd {

// defined in collide_ilp.hip, collide_ilp3.hip, collide_fp64.hip,
// collide_fp64_timed.hip and collide_generic_aux.hip
extern template __global__ void collide_batched<float, 4, false, false, true, kEitherLimit>(
    CollideArgs A);
extern template __global__ void collide_batched<float, 4, false, true, true, kEitherLimit>(
    CollideArgs A);
extern template __global__ void collide_batched<float, 4, true, false, false, kTimeLimited>(
    CollideArgs A);
extern template __global__ void collide_batched<float, 4, true, false, true, kTimeLimited>(
    CollideArgs A);
extern template __global__ void collide_batched<float, 4, true, false, false, kFixedCount>(
    CollideArgs A);
extern template __global__ void collide_batched<double, 4, false, false, false, kEitherLimit>(
    CollideArgs A);
extern template __global__ void collide_batched<double, 4, false, false, false, kFixedCount>(
    CollideArgs A);

template <typename Kern>
inline hipError_t prepare(Kern kern, size_t lds) {
  if (lds > 64 * 1024)
    return hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)lds);
  return hipSuccess;
}

template <typename RT, int KMAX, bool FAST, bool PROB>
inline hipError_t run_batched(const CollideArgs &a, int n_cells, int grid_override, hipStream_t s) {
  const size_t lds = std::max(region_bytes<RT>(a.big_cap, 4), 4 * region_bytes<RT>(a.small_cap, 1));
  // the composition mix and the event log only where they are used
  const bool aux = (a.comp != nullptr && a.P.n_comp > 0) || a.evlog != nullptr;
  const bool timed = a.dt > 0.0;
  auto kern = aux ? collide_batched<RT, KMAX, FAST, PROB, true>
                  : collide_batched<RT, KMAX, FAST, PROB, false>;
  // the mixed form's fast path and the FP64 form (up to 4 slots per lane)
  // come for one event budget only: without waiting times for fixed counts,
  // and (mixed) without the test for them in time-limited steps
  if constexpr (KMAX == 4 && !PROB && (sizeof(RT) == 8 || FAST))
    if (!aux && !timed) kern = collide_batched<RT, KMAX, FAST, PROB, false, kFixedCount>;
  if constexpr (KMAX == 4 && !PROB && sizeof(RT) == 4 && FAST)
    if (timed)
      kern = aux ? collide_batched<RT, KMAX, FAST, PROB, true, kTimeLimited>
                 : collide_batched<RT, KMAX, FAST, PROB, false, kTimeLimited>;
  hipError_t e = prepare(kern, lds);
  int dev = 0, cus = 0, per_cu = 0;
  if (e == hipSuccess) e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e == hipSuccess)
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)kern, 256, lds);
  if (e != hipSuccess) return e;
  if (per_cu < 1) return hipErrorInvalidConfiguration;
  // persistent workgroups: as many as fit, and no more than cells (the list
  // lengths are on the device; workgroups beyond the work exit at their first
  // queue pop, but starting them costs: a call over 8 cells takes 43 us with 8
  // workgroups, 73 with 768)
  int grid = std::min(per_cu * cus, std::max(n_cells, 1));
  if (grid_override > 0) grid = grid_override;
  CollideArgs b = a;
  b.seeded = grid <= per_cu * cus ? 1 : 0;
  kern<<<grid, 256, lds, s>>>(b);
  return hipGetLastError();
}

template <typename RT, int KMAX, bool FAST, bool PROB>
inline hipError_t run_plain(const CollideArgs &a, int n_cells, hipStream_t s) {
  const size_t lds = region_bytes<RT>(a.big_cap, 4);
  auto kern = collide_plain<RT, KMAX, FAST, PROB>;
  hipError_t e = prepare(kern, lds);
  if (e != hipSuccess) return e;
  if (n_cells > 0) kern<<<n_cells, 256, lds, s>>>(a);
  return hipGetLastError();
}

// the FP32 fast pair path applies to the physical kernel with all five
// velocity sources (the benchmark disk); everything else takes the generic one
inline bool fast_path(const CollideArgs &a, int precision) {
  const uint32_t all = DV_BROWNIAN | DV_TURB | DV_RADIAL | DV_AZIMUTHAL | DV_SETTLING;
  return precision != 0 && a.P.kernel == K_PHYSICAL && (a.P.flags & all) == all;
}

template <bool PROB>
hipError_t launch_batched(const CollideArgs &a, int precision, int n_cells, bool wide,
                          int grid_override, hipStream_t s);
template <bool PROB>
hipError_t launch_plain(const CollideArgs &a, int precision, int n_cells, bool wide, hipStream_t s);
template <>
hipError_t launch_batched<false>(const CollideArgs &, int, int, bool, int, hipStream_t);
template <>
hipError_t launch_batched<true>(const CollideArgs &, int, int, bool, int, hipStream_t);
template <>
hipError_t launch_plain<false>(const CollideArgs &, int, int, bool, hipStream_t);
template <>
hipError_t launch_plain<true>(const CollideArgs &, int, int, bool, hipStream_t);

template <bool PROB>
hipError_t batched_forms(const CollideArgs &a, int precision, int n_cells, bool wide,
                         int grid_override, hipStream_t s) {
  const bool fast = fast_path(a, precision);
  if (precision == 0)
    return wide ? run_batched<double, 8, false, PROB>(a, n_cells, grid_override, s)
                : run_batched<double, 4, false, PROB>(a, n_cells, grid_override, s);
  if (fast)
    return wide ? run_batched<float, 8, true, PROB>(a, n_cells, grid_override, s)
                : run_batched<float, 4, true, PROB>(a, n_cells, grid_override, s);
  return wide ? run_batched<float, 8, false, PROB>(a, n_cells, grid_override, s)
              : run_batched<float, 4, false, PROB>(a, n_cells, grid_override, s);
}

template <bool PROB>
hipError_t plain_forms(const CollideArgs &a, int precision, int n_cells, bool wide, hipStream_t s) {
  const bool fast = fast_path(a, precision);
  if (precision == 0)
    return wide ? run_plain<double, 8, false, PROB>(a, n_cells, s)
                : run_plain<double, 4, false, PROB>(a, n_cells, s);
  if (fast)
    return wide ? run_plain<float, 8, true, PROB>(a, n_cells, s)
                : run_plain<float, 4, true, PROB>(a, n_cells, s);
  return wide ? run_plain<float, 8, false, PROB>(a, n_cells, s)
              : run_plain<float, 4, false, PROB>(a, n_cells, s);
}

}  // namespace mcd
