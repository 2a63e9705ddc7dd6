// collide_device.hpp -- the per-cell collision Monte Carlo of the representative-
// particle method (Zsom & Dullemond 2008, adopted by the paper, Summary):
// build the row sums r_i = sum_j r_ij of the cell's rate matrix, then repeat
// events: exponential waiting time from the total rate R, choose i by the
// cumulative row sums, choose j by the cumulative rates of row i, apply the
// outcome (sticking / erosion / fragmentation) to i only, update every row
// sum incrementally for the changed particle and recompute row i.
//
// A cell is processed by a team of nw waves (1, or 4 for cells above the
// single-wave threshold, 256 particles by default); the two team shapes are
// separate instantiations of the cell body.  The cell's n particles are in
// canonical order j = 0..n-1; team lane t owns the contiguous slots
// j = t*K .. t*K+K-1 (K = ceil(n/(64 nw))), so the cumulative rate of j is the
// team prefix of the lanes' partial sums plus a short in-lane prefix.  Prefix
// sums are FP64 DPP scans in both forms; four-wave teams exchange wave totals
// through LDS (one barrier per scan).  A selection is made by the wave whose
// prefix range holds the target -- every wave finds it from the exchanged
// totals -- and published with one more barrier.  The uniforms of 64 events
// are drawn at once, one event per lane.  Particle records live in LDS as
// packed vectors indexed by s = q*64nw + t (slot q of lane t), so a wave reads
// consecutive 16-byte words.  Row sums (FP64), the per-event row values,
// masses and particle indices stay in registers of the owning lane; masses go
// back to HBM once, when the cell is done.  The starting row sums evaluate each
// unordered pair once (build_rows_pairwise*) in the FP32 fast path and in FP64,
// both up to four slots per lane; otherwise, and in FP64 teams of few particles,
// every row is summed in canonical order.  The batched kernel carries the composition mix and the event log only
// in the variant launched for runs that use them.
//
// The cell body and the kernel templates; collide_launch.hpp launches them.
#pragma once

#include <algorithm>

#include "device_common.hpp"
#include "internal.hpp"

namespace mcd {

// ---------------------------------------------------------------------------
// packed LDS records
// ---------------------------------------------------------------------------
template <typename RT>
struct RecStore;

// FP32: the three 16-byte words of a record lie together, so that one address
// serves all of a lane's slots (the slot and the word are immediate offsets);
// at a stride of 48 bytes the 16-byte reads of 16 consecutive lanes fall on
// distinct banks
template <>
struct RecStore<float> {
  float4 *D;  // per slot: (im, a, St, h) (q1, vr, vp, vz) (nd, m, ist, Mn)
  __device__ RecStore(char *base, int) : D((float4 *)base) {}
  __device__ Rec<float> load(int s) const {
    const float4 a = D[3 * s], b = D[3 * s + 1], c = D[3 * s + 2];
    Rec<float> r;
    r.im = a.x; r.a = a.y; r.St = a.z; r.h = a.w;
    r.q1 = b.x; r.vr = b.y; r.vp = b.z; r.vz = b.w;
    r.nd = c.x; r.m = c.y; r.ist = c.z; r.Mn = c.w;
    return r;
  }
  __device__ void store(int s, const Rec<float> &r) const {
    D[3 * s] = make_float4(r.im, r.a, r.St, r.h);
    D[3 * s + 1] = make_float4(r.q1, r.vr, r.vp, r.vz);
    D[3 * s + 2] = make_float4(r.nd, r.m, r.ist, r.Mn);
  }
};

// FP64: nine of the record's values, in four arrays of pairs and one of
// singles.  1 / (1 + St), which only pairs of large Stokes numbers read, is
// formed again by the same division, and 1 / St is not read by the FP64 pair
// rate: 72 bytes a particle let two workgroups of four 256-particle cells run
// on a CU (batched FP64 workload: 4.32 against 5.24 ms), 96 bytes one
template <>
struct RecStore<double> {
  double2 *D;  // (im, a) (St, h) (vr, vp) (vz, nd)
  double *E;   // m
  int cap;
  __device__ RecStore(char *base, int cap_)
      : D((double2 *)base), E((double *)((double2 *)base + 4 * cap_)), cap(cap_) {}
  __device__ Rec<double> load(int s) const {
    const double2 a = D[s], b = D[cap + s], c = D[2 * cap + s], d = D[3 * cap + s];
    Rec<double> r;
    r.im = a.x; r.a = a.y; r.St = b.x; r.h = b.y; r.vr = c.x; r.vp = c.y;
    r.vz = d.x; r.nd = d.y; r.m = E[s];
    r.q1 = 1.0 / (1.0 + r.St);
    r.ist = 0.0;  // not read
    r.Mn = 0.0;   // not held: the FP64 state is rebuilt from M
    return r;
  }
  __device__ void store(int s, const Rec<double> &r) const {
    D[s] = make_double2(r.im, r.a);
    D[cap + s] = make_double2(r.St, r.h);
    D[2 * cap + s] = make_double2(r.vr, r.vp);
    D[3 * cap + s] = make_double2(r.vz, r.nd);
    E[s] = r.m;
  }
};

// record of an empty slot: zero number density, so every rate against it
// vanishes; finite values elsewhere
template <typename RT>
__device__ inline Rec<RT> empty_rec() {
  Rec<RT> r;
  r.m = r.im = r.St = r.ist = (RT)1;
  r.a = r.h = r.vr = r.vp = r.vz = r.nd = r.Mn = (RT)0;
  r.q1 = (RT)0.5;
  return r;
}

// both directed rates of a pair and the relative velocity; inlined without
// exception (the one kernel of thirty in which the compiler called it instead
// passed the records through memory: row sums of 200 cells of 263 - 1024
// particles 6630 us instead of 1000)
template <typename RT, bool FAST>
struct PairEval {
  __device__ static __forceinline__ void run(const PairConst<RT> &c, const Rec<RT> &x, const Rec<RT> &y, RT &dv,
                             RT &rxy, RT &ryx) {
    const RT K = pair_kernel(c, x, y, dv);
    swarm_rates(c, x, y, K, rxy, ryx);
  }
};
template <>
struct PairEval<float, true> {
  __device__ static __forceinline__ void run(const PairConst<float> &c, const Rec<float> &x, const Rec<float> &y,
                             float &dv, float &rxy, float &ryx) {
    pair_rates_all(c, x, y, dv, rxy, ryx);
  }
};

// two partner sums on their way to another wave
template <typename RT>
struct alignas(2 * sizeof(RT)) Pair2 {
  RT x, y;
};
__device__ inline void build_pair(const PairConst<float> &c, const Rec<float> &x,
                                  const Rec<float> &y, float &rxy, float &ryx) {
  float dv;
  pair_rates_all<true>(c, x, y, dv, rxy, ryx);
}
__device__ inline void build_pair(const PairConst<double> &c, const Rec<double> &x,
                                  const Rec<double> &y, double &rxy, double &ryx) {
  double dv;
  PairEval<double, false>::run(c, x, y, dv, rxy, ryx);
}

// ---------------------------------------------------------------------------
// row sums of a one-wave cell, each unordered pair evaluated once
// ---------------------------------------------------------------------------
// Lane l holds slots (q, l), q < K.  Step 0 pairs the lane's own slots; step
// d = 1..32 pairs lane l with lane (l + d) mod 64 (at d = 32 only lanes below
// 32 evaluate, so every pair of lanes meets once).  r_xy goes to the lane's
// own sums; r_yx to an accumulator of the partner lane's sums that moves one
// lane down after every step (DPP wave rotation), so that the accumulator of
// lane X is always held by the lane currently paired with X; after step 32 it
// sits at lane X - 32 and returns with one exchange of the wave's halves.
// Sums are in the rate precision, in an order that differs from the members';
// slots past the cell's particles get 0.  In FP64, where a step takes longest, a
// cell of at most 32 lanes ends after the step of its last pair of lanes (the
// further steps add zeros).
template <typename RT, int KMAX>
__device__ inline void build_rows_pairwise(const RecStore<RT> &R, const PairConst<RT> &pc,
                                           int K, int lane, int n, double r[KMAX]) {
  const int steps = sizeof(RT) == 8 ? min(32, (n + K - 1) / K - 1) : 32;
  Rec<RT> mine[KMAX];
  RT acc[KMAX], pacc[KMAX];
#pragma unroll
  for (int q = 0; q < KMAX; ++q) {
    acc[q] = (RT)0;
    pacc[q] = (RT)0;
    if (q < K) mine[q] = R.load(q * 64 + lane);
  }
#pragma unroll
  for (int I = 0; I < KMAX; ++I) {
#pragma unroll
    for (int J = I; J < KMAX; ++J) {
      if (J < K) {
        RT rxy, ryx;
        build_pair(pc, mine[I], mine[J], rxy, ryx);
        acc[I] += rxy;
        if (J != I) acc[J] += ryx;
      }
    }
  }
#pragma unroll 1
  for (int d = 1; d <= steps; ++d) {
    const int c = (lane + d) & 63;
    Rec<RT> pr[KMAX];
#pragma unroll
    for (int J = 0; J < KMAX; ++J)
      if (J < K) pr[J] = R.load(J * 64 + c);
    const bool take = d < 32 || lane < 32;
#pragma unroll
    for (int I = 0; I < KMAX; ++I) {
#pragma unroll
      for (int J = 0; J < KMAX; ++J) {
        if (I < K && J < K) {
          RT rxy, ryx;
          build_pair(pc, mine[I], pr[J], rxy, ryx);
          acc[I] += take ? rxy : (RT)0;
          pacc[J] += take ? ryx : (RT)0;
        }
      }
    }
    if (d < steps) {
#pragma unroll
      for (int J = 0; J < KMAX; ++J)  // lane l takes lane l + 1's accumulators
        pacc[J] = dpp_t<0x134, 0xf, 0xf>(pacc[J]);
    }
  }
#pragma unroll
  for (int q = 0; q < KMAX; ++q) {
    const RT home = sizeof(RT) == 8 ? __shfl(pacc[q], (lane - steps) & 63, 64)
                                    : __shfl_xor(pacc[q], 32, 64);
    r[q] = (q < K && lane * K + q < n) ? (double)(acc[q] + home) : 0.0;
  }
}

// Four-wave teams: the same scheme over the team's 256 lanes.  Wave a
// first pairs its own lanes as above; then in phases p = 1..3 it pairs lane
// l with lane (l + d) mod 64 of wave b = (a + p) mod 4, for d = 0..31 if
// a < b and d = 1..32 if a > b (the two waves of a pair split the 64 lane
// offsets between them).  After each phase the partner accumulators, which
// moved one lane per step as above, go to wave b through the exchange buffer
// in two rounds of two slots (a barrier after each write and before reuse).
template <typename RT, int KMAX>
__device__ inline void build_rows_pairwise_team(const RecStore<RT> &R, const PairConst<RT> &pc,
                                                int K, int wave, int lane, int n, Pair2<RT> *xbuf,
                                                double r[KMAX]) {
  static_assert(KMAX % 2 == 0, "partner sums go over in pairs of slots");
  constexpr int TL = 256;
  const int own = wave * 64;
  const bool mine_any = own * K < n;
  Rec<RT> mine[KMAX];
  RT acc[KMAX], pacc[KMAX];
#pragma unroll
  for (int q = 0; q < KMAX; ++q) {
    acc[q] = (RT)0;
    pacc[q] = (RT)0;
    if (q < K) mine[q] = R.load(q * TL + own + lane);
  }
#pragma unroll
  for (int I = 0; I < KMAX; ++I) {
#pragma unroll
    for (int J = I; J < KMAX; ++J) {
      if (J < K) {
        RT rxy, ryx;
        build_pair(pc, mine[I], mine[J], rxy, ryx);
        acc[I] += rxy;
        if (J != I) acc[J] += ryx;
      }
    }
  }
  // the other lanes of the own wave
#pragma unroll 1
  for (int d = 1; d <= 32; ++d) {
    const int c = (lane + d) & 63;
    Rec<RT> pr[KMAX];
#pragma unroll
    for (int J = 0; J < KMAX; ++J)
      if (J < K) pr[J] = R.load(J * TL + own + c);
    const bool take = d < 32 || lane < 32;
#pragma unroll
    for (int I = 0; I < KMAX; ++I) {
#pragma unroll
      for (int J = 0; J < KMAX; ++J) {
        if (I < K && J < K) {
          RT rxy, ryx;
          build_pair(pc, mine[I], pr[J], rxy, ryx);
          acc[I] += take ? rxy : (RT)0;
          pacc[J] += take ? ryx : (RT)0;
        }
      }
    }
    if (d < 32) {
#pragma unroll
      for (int J = 0; J < KMAX; ++J)
        pacc[J] = dpp_t<0x134, 0xf, 0xf>(pacc[J]);
    }
  }
#pragma unroll
  for (int q = 0; q < KMAX; ++q) {
    acc[q] += __shfl_xor(pacc[q], 32, 64);
    pacc[q] = (RT)0;
  }
  // the lanes of the other three waves
#pragma unroll 1
  for (int p = 1; p <= 3; ++p) {
    const int b = (wave + p) & 3;
    const int d0 = wave < b ? 0 : 1;
    // (FP64, where a step takes longest: none against or of an empty wave, which
    // would add zeros)
    const int n_st = sizeof(RT) == 4 || (mine_any && b * 64 * K < n) ? 32 : 0;
#pragma unroll 1
    for (int st = 0; st < n_st; ++st) {
      const int c = (lane + d0 + st) & 63;
      Rec<RT> pr[KMAX];
#pragma unroll
      for (int J = 0; J < KMAX; ++J)
        if (J < K) pr[J] = R.load(J * TL + b * 64 + c);
#pragma unroll
      for (int I = 0; I < KMAX; ++I) {
#pragma unroll
        for (int J = 0; J < KMAX; ++J) {
          if (I < K && J < K) {
            RT rxy, ryx;
            build_pair(pc, mine[I], pr[J], rxy, ryx);
            acc[I] += rxy;
            pacc[J] += ryx;
          }
        }
      }
      if (st < 31) {
#pragma unroll
        for (int J = 0; J < KMAX; ++J)
          pacc[J] = dpp_t<0x134, 0xf, 0xf>(pacc[J]);
      }
    }
    // lane l now holds the sums of lane (l + d0 + 31) mod 64 of wave b; they
    // go over in two rounds of two slots
#pragma unroll
    for (int h = 0; h < KMAX; h += 2) {
      xbuf[b * 64 + ((lane + d0 + 31) & 63)] = Pair2<RT>{pacc[h], pacc[h + 1]};
      block_lds_sync();
      const Pair2<RT> in = xbuf[own + lane];
      acc[h] += in.x;
      acc[h + 1] += in.y;
      block_lds_sync();
    }
#pragma unroll
    for (int q = 0; q < KMAX; ++q) pacc[q] = (RT)0;
  }
  const int tl = own + lane;
#pragma unroll
  for (int q = 0; q < KMAX; ++q) r[q] = (q < K && tl * K + q < n) ? (double)acc[q] : 0.0;
}

// Four-wave teams with one slot per lane at most: every row over the n members in
// their order.  The 128 steps of the scheme above take as long as 192 members
// here (FP64, physical kernel: one cell of 64 / 192 / 256 particles 36 / 96 / 113
// us against 97, 3000 cells of 128 / 192 / 256 494 / 758 / 1031 against 641)
constexpr int kPlainRows = 192;
template <typename RT, int KMAX>
__device__ inline void build_rows_plain(const RecStore<RT> &R, const PairConst<RT> &pc, int tl,
                                        int n, double r[KMAX]) {
  const Rec<RT> mine = R.load(tl);
  RT acc = (RT)0;
  for (int k = 0; k < n; ++k) {
    RT dv, rxy, ryx;
    PairEval<RT, false>::run(pc, mine, R.load(k), dv, rxy, ryx);
    acc += rxy;
  }
#pragma unroll
  for (int q = 0; q < KMAX; ++q) r[q] = q == 0 && tl < n ? (double)acc : 0.0;
}

// ---------------------------------------------------------------------------
// team: the NW waves (1 or 4) that process a cell
// ---------------------------------------------------------------------------
template <int NW>
__device__ inline void team_sync() {
  if constexpr (NW > 1)
    block_lds_sync();
  else
    wave_lds_sync();
}

// Team-inclusive prefix of x over the team lanes and its total.  Teams of
// four waves exchange their totals through `slot` (one barrier); p[w] is then
// the prefix of the waves' totals up to wave w, added in wave order.
// With TWO, y is summed too: over each wave in its own precision (BT), then in
// FP64 over the waves, in the same exchange.
// A slot may be written again only after another barrier of the team.
template <int NW, bool TWO, typename BT>
__device__ __forceinline__ double team_scan(double x, BT y, int wave, int lane, double *slot, double p[4],
                                   double &tot_x, double &tot_y) {
  double inc = x;
  double wy = 0.0;
  if constexpr (TWO) {
    wave_incl_scan2(inc, y);
    wy = (double)readlane_t(y, 63);
  } else {
    inc = wave_incl_scan(inc);
  }
  const double wx = readlane_d(inc, 63);
  if constexpr (NW == 1) {
    tot_x = wx;
    if (TWO) tot_y = wy;
    return inc;
  } else {
    if (lane == 63) {
      slot[wave] = wx;
      if (TWO) slot[4 + wave] = wy;
    }
    block_lds_sync();
    const double2 a = ((const double2 *)slot)[0], b = ((const double2 *)slot)[1];
    p[0] = a.x;
    p[1] = p[0] + a.y;
    p[2] = p[1] + b.x;
    p[3] = p[2] + b.y;
    tot_x = p[3];
    if (TWO) {
      const double2 c = ((const double2 *)slot)[2], d = ((const double2 *)slot)[3];
      tot_y = ((c.x + c.y) + d.x) + d.y;
    }
    const double off = wave == 0 ? 0.0 : (wave == 1 ? p[0] : (wave == 2 ? p[1] : p[2]));
    return off + inc;
  }
}

// particle state after a collision: FP64 formulas for the FP64 path, the
// FP32 formulas with per-cell FP32 factors for the mixed path
template <typename RT>
struct RecAfter;
template <>
struct RecAfter<double> {
  __device__ static Rec<double> get(const Model &P, const TeamScratch *S, const CellF &, double m,
                                    double M, double) {
    return make_rec<double>(P, S->gas, m, M, 1.0);
  }
};
template <>
struct RecAfter<float> {
  __device__ static Rec<float> get(const Model &, const TeamScratch *, const CellF &cf, double m,
                                   double, float Mn) {
    return make_rec_f(cf, m, Mn);
  }
};

// ---------------------------------------------------------------------------
// selection: the first slot whose cumulative value exceeds a target
// ---------------------------------------------------------------------------
// Search inside one wave.  v[] are the lane's K values in canonical order,
// part their sum, incl the team-inclusive prefix of part.  ql is the lane's
// first slot whose running sum exceeds the target (K if none does); the
// chosen lane src is the first that has such a slot and a nonzero partial.
// Every lane searches its own slots as if it owned the pick, so the search
// does not wait for the choice of the lane; false if no lane has a hit.
template <int KC, typename VT>
__device__ __forceinline__ bool wave_search(double incl, double part, const VT *v, int K, double target,
                                   uint64_t go, int &src, int &ql) {
  double c[KC];
  double cum = incl - part;
#pragma unroll
  for (int q = 0; q < KC; ++q) {
    if (q < K) cum += (double)v[q];
    c[q] = cum;
  }
  ql = KC - 1;
#pragma unroll
  for (int q = KC - 2; q >= 0; --q) ql = c[q] > target ? q : ql;
  // masks, not conditions, are combined: a ballot of one compare is the
  // compare itself
  const uint64_t hit = ballot(part > 0.0) & ballot(c[KC - 1] > target) & go;
  src = __builtin_ctzll(hit | (1ull << 63));
  return hit != 0;
}

// Where rounding leaves no lane of the wave past the target: its last lane
// with a nonzero partial, and there the last nonzero slot; false if every
// partial is zero.
template <int KC, typename VT>
__device__ __forceinline__ bool wave_last(double part, const VT *v, int K, int &src, int &ql) {
  const uint64_t pos = ballot(part > 0.0);
  src = 63 - __builtin_clzll(pos | 1ull);
  ql = 0;
#pragma unroll
  for (int q = 0; q < KC; ++q)
    if (q < K) ql = v[q] > (VT)0 ? q : ql;
  return pos != 0;
}

// slot ql (per lane) of the lane's values
template <int KC, typename T>
__device__ __forceinline__ T lane_pick(const T *a, int ql) {
  T x = a[0];
#pragma unroll
  for (int q = 1; q < KC; ++q) {
    const T v = a[q];  // a value, not a choice of addresses: the array stays in registers
    x = ql == q ? v : x;
  }
  return x;
}

// The wave of a four-wave team that holds the target: the first whose prefix
// p[w] (plus delta from wave fix_wave on) exceeds it.  Every wave has the same
// prefixes and finds the same owner without another exchange.  -1 if none.
__device__ __forceinline__ int owner_wave(const double p[4], double target, int fix_wave, double delta) {
  const uint64_t b0 = ballot((fix_wave <= 0 ? p[0] + delta : p[0]) > target);
  const uint64_t b1 = ballot((fix_wave <= 1 ? p[1] + delta : p[1]) > target);
  const uint64_t b2 = ballot((fix_wave <= 2 ? p[2] + delta : p[2]) > target);
  const uint64_t b3 = ballot((fix_wave <= 3 ? p[3] + delta : p[3]) > target);
  return b0 ? 0 : (b1 ? 1 : (b2 ? 2 : (b3 ? 3 : -1)));
}

// A pick as every lane of the team knows it: the chosen slot s (its index in
// the record store, -1: nothing to pick), the particle's mass m, the chosen
// value x (row sum of i, relative velocity of j).
template <typename XT>
struct Picked {
  double m;
  XT x;
  int s;
};

// One-wave pick of the chosen slot's values by lane reads.
template <int KC, typename XT>
__device__ __forceinline__ Picked<XT> read_pick(int src, int ql, const double *m, const XT *x) {
  Picked<XT> o;
  const int qs = readlane_i(ql, src);
  o.s = qs * 64 + src;
  o.m = readlane_d(lane_pick<KC>(m, ql), src);
  o.x = readlane_t(lane_pick<KC>(x, ql), src);
  return o;
}

// The chosen lane of a four-wave team publishes its slot: the owner wave's
// search, or where rounding leaves no lane past the target its last lane with
// a nonzero partial (slot -1: there is none either) ...
template <int KC, typename XT>
__device__ __forceinline__ void write_pick(TeamCand *C, int wave, int lane, int src, int ql, bool any,
                                           const double *m, const XT *x) {
  if (lane == src) {
    C->m = lane_pick<KC>(m, ql);
    if constexpr (sizeof(XT) == 4)
      C->xf = lane_pick<KC>(x, ql);
    else
      C->x = lane_pick<KC>(x, ql);
    C->s = any ? ql * 256 + wave * 64 + lane : -1;
  }
}
template <int KC, typename XT, typename VT>
__device__ __forceinline__ void publish_pick(TeamCand *C, int wave, int lane, double incl,
                                             double part, const VT *v, int K, double target,
                                             const double *m, const XT *x) {
  int src, ql;
  bool any = true;
  if (!wave_search<KC>(incl, part, v, K, target, ~0ull, src, ql))
    any = wave_last<KC>(part, v, K, src, ql);
  write_pick<KC, XT>(C, wave, lane, src, ql, any, m, x);
}
// ... and every lane reads it after the barrier.
template <typename XT>
__device__ __forceinline__ Picked<XT> fetch_pick(const TeamCand *C) {
  Picked<XT> o;
  o.m = C->m;
  if constexpr (sizeof(XT) == 4)
    o.x = C->xf;
  else
    o.x = C->x;
  o.s = __builtin_amdgcn_readfirstlane(C->s);
  return o;
}

// Team pick where the owner found no hit (or rounding left no owner): every
// wave searches; the first wave with a hit wins, else the last wave with any
// nonzero partial.  s < 0: every partial is zero.
template <int KC, typename VT, typename XT>
__device__ __forceinline__ Picked<XT> pick_all_waves(TeamScratch *S, TeamCand *C, int wave, int lane,
                                            double incl, double part, const VT *v, int K,
                                            double target, const double *m, const XT *x) {
  int src, ql;
  int code = wave_search<KC>(incl, part, v, K, target, ~0ull, src, ql) ? 2 : 0;
  if (code == 0) code = wave_last<KC>(part, v, K, src, ql) ? 1 : 0;
  if (lane == 0) S->code[wave] = code;
  block_lds_sync();
  int wsel = -1;
  for (int w = 3; w >= 0; --w)
    if (S->code[w] == 2) wsel = w;
  if (wsel < 0)
    for (int w = 0; w < 4; ++w)
      if (S->code[w] == 1) wsel = w;
  if (wave == wsel) write_pick<KC, XT>(C, wave, lane, src, ql, true, m, x);
  block_lds_sync();
  Picked<XT> o = fetch_pick<XT>(C);
  if (wsel < 0) o.s = -1;
  block_lds_sync();  // the codes and the candidate are read before they are written again
  return o;
}

// Outcome of an event for i (mass mi) hitting a body of swarm j (mass mj) at
// relative velocity dv: the new mass, and the counts of the rarer outcomes.
// fast: the collision fragments or erodes.  The FP64 form takes it from
// outcome(); the mixed form computes the sticking and the eroding mass side by
// side with its division-free equivalents (no branch on the common outcomes)
// and enters a branch only for the fragment draws.  n_fast counts erosions
// too.  Returns the outcome code where CODE asks for it.
struct OutcomeCounts {
  uint32_t n_fast = 0, n_small = 0, n_frag = 0;
};
template <typename RT, bool CODE>
__device__ __forceinline__ int event_outcome(const OutcomeConst &P, bool fast, double mi, double mj,
                                             double u4, double &mnew, OutcomeCounts &n) {
  if constexpr (sizeof(RT) == 8) {
    const int oc = __builtin_amdgcn_readfirstlane(outcome(P, fast, mi, mj, u4, mnew));
    n.n_fast += oc != OUT_STICK ? 1u : 0u;
    n.n_small += oc == OUT_ERODED_SMALL ? 1u : 0u;
    n.n_frag += oc == OUT_FRAG ? 1u : 0u;
    return oc;
  } else {
    const double d = P.dm_max * mi;
    const double gm = (P.dm_max > 0.0 && d > mj) ? d : mj;
    const double er = mi - P.erosion_chi * gm;
    const double ec = er > P.m0 ? er : P.m0;
    const double big = mi > mj ? mi : mj, small = mi > mj ? mj : mi;
    const uint64_t mf = ballot(fast);
    const uint64_t uneven = ballot(big >= P.erosion_ratio * small);
    mnew = fast ? ec : mi + gm;
    int oc = OUT_STICK;
    if (CODE) oc = mf ? OUT_ERODE : OUT_STICK;
    n.n_fast += mf ? 1u : 0u;
    if (mf & ~(uneven & ballot(mi >= mj))) {
      mnew = frag_draw(P.m0, uneven ? mi : big, u4);
      n.n_small += uneven ? 1u : 0u;
      n.n_frag += uneven ? 0u : 1u;
      if (CODE) oc = uneven ? OUT_ERODED_SMALL : OUT_FRAG;
    }
    return oc;
  }
}

// Composition of i after a sticking or fragmenting event: mass-weighted mix
// of i's fractions (weight m_i) and j's (weight g m_j), one component per
// lane below n_comp.  The fractions are loaded as soon as i and j are known
// (comp_load) and the mix is stored early in the next event, once its i is
// chosen, or when the cell ends (comp_store): the loads then have the rest of
// the event and the next event's selection of i to arrive instead of
// stalling the chain.  The next event's own loads come after that store, and
// a load of a lane after its own store to the same address reads the store.
struct CompMix {
  float cI, cJ;
  bool on;
};
__device__ inline CompMix comp_load(const CollideArgs &A, int lane, bool writer, int gi, int gj) {
  CompMix c{0.0f, 0.0f, false};
  if (writer && A.comp != nullptr && lane < A.P.n_comp) {
    // the component's base is formed here, per event, not held (or spilled)
    // across the event loop
    const float *cs = A.comp + (size_t)opaque_v(lane) * A.N;
    c.cI = cs[gi];
    c.cJ = cs[gj];
    c.on = true;
  }
  return c;
}
template <bool EXACT>
__device__ inline void comp_store(const CollideArgs &A, const CompMix &c, int lane, int oc, int gi,
                                  double mi, double mj) {
  if (c.on && (oc == OUT_STICK || oc == OUT_FRAG)) {
    // the grouped mass g m_j as the outcome formed it
    double wj;
    if (EXACT) {
      wj = group_factor(A.P.dm_max, mi, mj) * mj;
    } else {
      const double d = A.P.dm_max * mi;
      wj = (A.P.dm_max > 0.0 && d > mj) ? d : mj;
    }
    A.comp[(size_t)opaque_v(lane) * A.N + gi] =
        (float)((mi * (double)c.cI + wj * (double)c.cJ) / (mi + wj));
  }
}

__device__ inline void log_event(const CollideArgs &A, int cell, uint32_t e, int i_local,
                                 int j_local, int oc) {
  if (A.evlog != nullptr && (int64_t)e < A.log_per_cell) {
    int32_t *L = A.evlog + ((size_t)cell * A.log_per_cell + e) * 4;
    L[0] = i_local;
    L[1] = j_local;
    L[2] = oc;
    L[3] = 0;
  }
}

// the event budget a kernel is compiled for: a fixed number of events per
// cell (dt = 0), a time limit dt > 0, or either, read from the arguments
enum : int { kFixedCount = 0, kTimeLimited = 1, kEitherLimit = 2 };

// ---------------------------------------------------------------------------
// the events of one cell
// ---------------------------------------------------------------------------
// KC: slots per lane; with FIXED every lane of the team has exactly KC slots
// (K == KC), otherwise K <= KC of them.  AUX: the composition mix and the event
// log are compiled in (a launch with fractions to track or events to record);
// without them the event loop carries neither.  LIMIT: a kernel compiled for
// fixed counts only carries no waiting times (their logarithm, the time test,
// the priority rule).
//
// A cell's events are one serial chain, and beyond the 2 K pair evaluations its
// length is that of an event's control: what the chain waits for counts, not
// the number of instructions alone.  Hence: the slots per lane are a
// compile-time number (no branch per slot, one block whose loads and pairs
// interleave); the tests that end a cell (time limit, vanished total) are part
// of the selection's ballot, one branch for all of them; a chosen slot's values
// are selected per lane while the chosen lane is still being found; the
// outcome's and the new record's parameters are read from LDS while row i is
// evaluated; the common outcomes are computed without a branch; the rare
// cases (rounding left no hit, row i without a partner) join the common path
// instead of leaving the loop body by an exit of their own.
template <typename RT, int KC, bool FIXED, bool FAST, bool PROB, bool AUX, int NW, int LIMIT>
__device__ __forceinline__ void run_events(const CollideArgs &A, const PairConst<RT> &pc,
                                           const RecStore<RT> &R, TeamScratch *S, int cell, int s0,
                                           int n, int K_cell, double scale, int wave_cell,
                                           int lane_cell, uint32_t step, double *r, double *m64) {
  constexpr int TL = 64 * NW;
  // the records of all slots are requested before the first pair: one wait on
  // LDS per pass instead of one per slot (a lone cell of 200 particles: 1.84
  // against 1.94 us per event)
  constexpr bool AHEAD = FIXED && KC > 1 && sizeof(RT) == 4;
  const bool timed = LIMIT == kEitherLimit ? A.dt > 0.0 : LIMIT == kTimeLimited;
  const uint32_t emax = A.max_events > 0 ? (uint32_t)A.max_events : 0xFFFFFFFFu;
  const uint32_t c32 = (uint32_t)cell;
  uint32_t e = 0;  // events so far (fewer than 2^32 per cell and step)
  uint32_t n_null = 0;
  OutcomeCounts cnt;
  uint64_t bad_mass = 0;
  // slots that hold a particle, as lane masks
  uint64_t valid[KC];
#pragma unroll
  for (int q = 0; q < KC; ++q) {
    const int K = FIXED ? KC : K_cell;
    valid[q] = ballot(q < K && (wave_cell * 64 + lane_cell) * K + q < n);
  }
  // what the previous event leaves to the next scan: the wave-partial new row
  // sum of its i, i's old row sum and its place (own[q]: its lane, if its slot
  // is q; own_lane: its team lane).  None before the first event, and none for
  // a scan repeated on the row sums as they are
  RT part2 = (RT)0;
  double ri_old = 0.0;
  int own_lane = TL;
  uint64_t own[KC];
#pragma unroll
  for (int q = 0; q < KC; ++q) own[q] = 0;
  double t = 0.0, Rtot = 0.0;
  // uniforms of 64 consecutive events: lane l holds -ln u1, u2, u3, u4 of
  // event e0 + l from Philox(e0 + l, cell, step, 0) and (.., 1)
  double nlu1 = 0.0, uu2 = 0.0, uu3 = 0.0, uu4 = 0.0, uu5 = 0.0;
  int rl = 0, rl_end = 0;  // the event's lane of that batch, and the batch's end
  // the previous event's composition mix, not yet stored
  CompMix pcm{0.0f, 0.0f, false};
  int p_oc = 0, p_gi = 0;
  double p_mi = 0.0, p_mj = 0.0;
  int si = 0;  // the chosen i: slot and mass (its old row sum is ri_old)
  double mi = 0.0;
  // what one choice of i passes along: prefix and lane sum of the row sums,
  // (four-wave teams) the waves' prefixes, their correction and the pick
  double incl = 0.0, part = 0.0, p[4], delta = 0.0, t_next = 0.0, target = 0.0;
  uint64_t go = 0;
  int src = 0, ql = 0;
  Picked<double> ci;

  // -- prefix of the row sums and the new r_i in one exchange.  The owner's
  // slot still holds the old r_i and is corrected here; in four-wave teams,
  // waves from i's on carry delta on top of the prefixes p[]
  auto scan_rows = [&](int K, int lane, int wave) __attribute__((always_inline)) {
    const int tl = wave * 64 + lane;
    part = r[0];  // K >= 1
#pragma unroll
    for (int q = 1; q < KC; ++q)
      if (FIXED || q < K) part += r[q];
    double ri_new;
    incl = team_scan<NW, true>(part, part2, wave, lane, S->tot_i, p, Rtot, ri_new);
    delta = ri_new - ri_old;
    incl += tl >= own_lane ? delta : 0.0;
    Rtot += delta;
    part += tl == own_lane ? delta : 0.0;
#pragma unroll
    for (int q = 0; q < KC; ++q)
      r[q] = __builtin_amdgcn_inverse_ballot_w64(own[q]) ? ri_new : r[q];
  };

  // the uniforms of the next 64 events, one event per lane
  auto draw = [&](int lane) __attribute__((always_inline)) {
    const uint32_t ec = e + (uint32_t)lane;
    // the key schedule is formed here, once per 64 events, not held
    const uint32_t k0 = opaque_u(A.P.key0), k1 = opaque_u(A.P.key1);
    const U4 w0 = philox4x32_10(U4{ec, c32, step, 0u}, k0, k1);
    const U4 w1 = philox4x32_10(U4{ec, c32, step, 1u}, k0, k1);
    if (timed) nlu1 = -log(u01(w0.x, w0.y));
    uu2 = u01(w0.z, w0.w);
    uu3 = u01(w1.x, w1.y);
    uu4 = u01(w1.z, w1.w);
    if constexpr (PROB) {  // the fragmentation uniform u5
      const U4 w3 = philox4x32_10(U4{ec, c32, step, 3u}, k0, k1);
      uu5 = u01(w3.x, w3.y);
    }
    rl = 0;
    rl_end = (int)(emax - e < 64u ? emax - e : 64u);
  };

  // the end of the exponential waiting time; the FP32 form takes 1/R from the
  // hardware estimate and one Newton step
  auto next_time = [&](double R) __attribute__((always_inline)) -> double {
    if (!timed) return t;
    if constexpr (sizeof(RT) == 4) {
      double ir = __builtin_amdgcn_rcp(R);
      ir = fma(fma(-R, ir, 1.0), ir, ir);
      return t + readlane_d(nlu1, rl) * ir * scale;
    } else {
      return t + readlane_d(nlu1, rl) / R * scale;
    }
  };

  // -- choose i by cumulative row sums; false: see choose_rare
  auto choose = [&](int K, int lane, int wave) __attribute__((always_inline)) -> bool {
    t_next = next_time(Rtot);
    go = ballot(Rtot > 0.0);
    if (timed) go &= ballot(!(t_next > A.dt));  // else the next event falls outside the step
    target = readlane_d(uu2, rl) * Rtot;
    if constexpr (NW == 1) {
      return wave_search<KC>(incl, part, r, K, target, go, src, ql);
    } else {
      const int ow = go ? owner_wave(p, target, own_lane >> 6, delta) : -1;
      if (wave == ow)
        publish_pick<KC, double>(&S->ci, wave, lane, incl, part, r, K, target, m64, r);
      block_lds_sync();
      ci = fetch_pick<double>(&S->ci);
      return (ow | ci.s) >= 0;
    }
  };
  // No hit, the time is over, or the running total vanished.  That total (the
  // scan plus the change of r_i) can round to zero while a row sum still holds
  // a positive remainder, and rounding can leave every prefix below the
  // target: the cell is done only when a fresh sum of the row sums is zero, as
  // in the method's definition of R.  false: the cell is done
  auto choose_rare = [&](int K, int lane, int wave) __attribute__((always_inline)) -> bool {
    const bool fresh = own_lane == TL;
    bool ok = false;
    if (NW > 1) block_lds_sync();
    if (ballot(Rtot > 0.0)) {
      if (ballot(isfinite(Rtot)) == 0 || go == 0) return false;
      if constexpr (NW == 1) {
        ok = wave_last<KC>(part, r, K, src, ql);
      } else {
        ci = pick_all_waves<KC, double, double>(S, &S->ci, wave, lane, incl, part, r, K,
                                                     target, m64, r);
        ok = ci.s >= 0;
      }
    }
    if (ok) return true;
    // a total of rounding remainders ends the cell; a positive fresh total
    // takes the event on the fresh prefixes
    if (!fresh) {
      part = r[0];
#pragma unroll
      for (int q = 1; q < KC; ++q)
        if (FIXED || q < K) part += r[q];
      double unused;
      incl = team_scan<NW, false>(part, 0.0f, wave, lane, S->tot_i, p, Rtot, unused);
      t_next = next_time(Rtot);
      if (ballot(Rtot > 0.0) == 0 || ballot(isfinite(Rtot)) == 0) return false;
      if (timed && ballot(t_next > A.dt)) return false;
      target = readlane_d(uu2, rl) * Rtot;
      if constexpr (NW == 1) {
        ok = wave_search<KC>(incl, part, r, K, target, ~0ull, src, ql) ||
             wave_last<KC>(part, r, K, src, ql);
      } else {
        block_lds_sync();
        ci = pick_all_waves<KC, double, double>(S, &S->ci, wave, lane, incl, part, r, K,
                                                     target, m64, r);
        ok = ci.s >= 0;
      }
    } else if (ballot(Rtot > 0.0) == 0) {
      return false;
    }
    if (!ok && wave * 64 + lane == 0) atomicOr(&A.state->flags, FLAG_BAD_RATE);
    return ok;
  };
  auto take = [&]() __attribute__((always_inline)) {
    if constexpr (NW == 1) ci = read_pick<KC, double>(src, ql, m64, r);
    t = t_next;
    si = ci.s;
    mi = ci.m;
    ri_old = ci.x;
  };

  bool any;
  {
    const int wave = NW == 1 ? 0 : wave_cell;
    scan_rows(K_cell, lane_cell, wave);
    if (timed) {
      // time-limited steps: a cell whose expected event count R dt is large is
      // a long serial chain that can outlast every other cell of the step, so
      // its waves get a higher issue priority on their SIMD (the rest fill in
      // around them); back to the default when the cell is done
      const double expect = Rtot / scale * A.dt;
      if (expect >= 256.0)
        __builtin_amdgcn_s_setprio(3);
      else if (expect >= 64.0)
        __builtin_amdgcn_s_setprio(2);
      else if (expect >= 16.0)
        __builtin_amdgcn_s_setprio(1);
    }
    draw(lane_cell);
    any = choose(K_cell, lane_cell, wave) || choose_rare(K_cell, lane_cell, wave);
  }
  // The scan and the choice of the next event's i stand at the end of the loop
  // body, after the update of the row sums, so that they are scheduled
  // together; the rare ways out leave the loop directly.
  if (any) for (;;) {
    take();
    // lane and wave indices (and K) per event: lane masks formed from them are
    // made where they are needed instead of being kept across the loop
    const int K = FIXED ? KC : opaque_s(K_cell);
    const int lane = opaque_v(lane_cell);
    const int wave = NW == 1 ? 0 : opaque_s(wave_cell);
    const int tl = wave * 64 + lane;
    if constexpr (AUX) {
      if (pcm.on) {
        comp_store<sizeof(RT) == 8>(A, pcm, lane, p_oc, p_gi, p_mi, p_mj);
        pcm.on = false;
      }
    }
    // particle indices are read from the cell order where an event needs them
    // (fractions; the FP64 state of i, rebuilt from its swarm mass): the loads
    // overlap the rows, and no register holds them through the events
    int gi = 0;
    double Mi = 0.0;
    if constexpr (AUX || sizeof(RT) == 8) gi = A.order[s0 + (si & (TL - 1)) * K + si / TL];
    if constexpr (sizeof(RT) == 8) Mi = A.M[gi];
    const Rec<RT> ri = R.load(si);

    Rec<RT> rq[KC];
    if constexpr (AHEAD) {
#pragma unroll
      for (int q = 0; q < KC; ++q) rq[q] = R.load(q * TL + tl);
      __builtin_amdgcn_sched_barrier(0);
    }
    // -- row i before the event: r_ij, r_ji and the relative velocities
    RT rij[KC], rji[KC], dvv[KC];
    double part1 = 0.0;
#pragma unroll
    for (int q = 0; q < KC; ++q) {
      rij[q] = (RT)0;
      rji[q] = (RT)0;
      dvv[q] = (RT)0;
      if (FIXED || q < K) {  // empty slots have zero density: rij = 0
        if constexpr (!AHEAD) rq[q] = R.load(q * TL + tl);
        PairEval<RT, FAST>::run(pc, ri, rq[q], dvv[q], rij[q], rji[q]);
      }
      part1 = q == 0 ? (double)rij[0] : part1 + (double)rij[q];
    }
    // the outcome's and the new record's parameters, read while the scan runs
    OutcomeConst oc_par;
    CellF cf;
    if constexpr (sizeof(RT) == 4) {
      oc_par = S->oc;
      cf = S->cf;
    }
    double Ri, pj[4];
    double unused;
    const double incl1 =
        team_scan<NW, false>(part1, 0.0f, wave, lane, S->tot_j, pj, Ri, unused);
    if constexpr (sizeof(RT) == 4) {
      asm volatile("" ::"v"(oc_par.dm_max), "v"(oc_par.erosion_chi), "v"(oc_par.erosion_ratio),
                   "v"(oc_par.m0), "v"(oc_par.v_frag));
      asm volatile("" ::"v"(cf.ca), "v"(cf.a_sw), "v"(cf.tE), "v"(cf.tS), "v"(cf.Om), "v"(cf.Ste),
                   "v"(cf.m2eta), "v"(cf.meta), "v"(cf.mzO));
    } else {
      oc_par = S->oc;
    }
    // row i may have no partner left (its stored sum was rounding residue):
    // a null event clears it.  It takes the common path with every update
    // masked out
    const bool null = ballot(Ri > 0.0) == 0;
    // -- choose j (its mass, relative velocity, index), then the outcome
    // (only i changes), computed alike by every wave
    const double target_j = readlane_d(uu3, rl) * Ri;
    Picked<RT> cj;
    if constexpr (NW == 1) {
      if (!wave_search<KC>(incl1, part1, rij, K, target_j, ~0ull, src, ql))
        wave_last<KC>(part1, rij, K, src, ql);
      cj = read_pick<KC, RT>(src, ql, m64, dvv);
    } else {
      const int ow = owner_wave(pj, target_j, NW, 0.0);
      if (wave == ow)
        publish_pick<KC, RT>(&S->cj, wave, lane, incl1, part1, rij, K, target_j, m64, dvv);
      block_lds_sync();
      cj = fetch_pick<RT>(&S->cj);
      if ((ow < 0 || cj.s < 0) && !null) {
        block_lds_sync();
        cj = pick_all_waves<KC, RT, RT>(S, &S->cj, wave, lane, incl1, part1, rij, K, target_j,
                                             m64, dvv);
      }
    }
    CompMix cm{0.0f, 0.0f, false};
    if constexpr (AUX)
      if (!null && A.comp != nullptr && wave == 0)
        cm = comp_load(A, lane, true, gi, A.order[s0 + (cj.s & (TL - 1)) * K + cj.s / TL]);
    bool fast;
    if constexpr (PROB) {
      fast = readlane_d(uu5, rl) < (double)frag_probability(oc_par, cj.x);
    } else {
      fast = !(cj.x < (RT)oc_par.v_frag);
    }
    if (null) {
      // a partner of i's own mass: nothing takes the outcome, but it has to be
      // a valid mass (of zero mass, the FP64 grouping factor would be infinite
      // and the outcome not a number)
      cj.m = mi;
      fast = false;
      ++n_null;
    }
    double mnew;
    const int oc = event_outcome<RT, AUX>(oc_par, fast, mi, cj.m, readlane_d(uu4, rl), mnew, cnt);
    bad_mass |= ballot(!(mnew > 0.0) || !isfinite(mnew));
    const Rec<RT> rin = RecAfter<RT>::get(A.P, S, cf, mnew, Mi, ri.Mn);
    if constexpr (AUX) {
      if (A.evlog != nullptr && tl == 0)
        log_event(A, cell, e, (si & (TL - 1)) * K + si / TL,
                  null ? -1 : (cj.s & (TL - 1)) * K + cj.s / TL, null ? -1 : oc);
    }
    // the owner of i keeps the new record and mass; it alone reads the slot
    // until the next exchange.  own[q]: its lane, if the slot is q
    const int qi = si / TL;
    own_lane = si & (TL - 1);
    const uint64_t own_bit = NW == 1 || wave == own_lane >> 6 ? 1ull << (si & 63) : 0ull;
#pragma unroll
    for (int q = 0; q < KC; ++q) own[q] = (KC == 1 || q == qi) ? own_bit : 0ull;
    if (__builtin_amdgcn_inverse_ballot_w64(null ? 0ull : own_bit)) R.store(si, rin);

    // -- new row i: incremental update of the other rows, fresh row sum of
    // i in the rate precision within a wave (the FP32 tree adds no more
    // than the rates' own rounding), then FP64
    part2 = (RT)0;
    if constexpr (AHEAD) {
#pragma unroll
      for (int q = 0; q < KC; ++q) rq[q] = R.load(q * TL + tl);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int q = 0; q < KC; ++q) {
      if (FIXED || q < K) {
        if constexpr (!AHEAD) rq[q] = R.load(q * TL + tl);
        RT dv, a_iq, a_qi;
        PairEval<RT, FAST>::run(pc, rin, rq[q], dv, a_iq, a_qi);
        part2 = q == 0 ? a_iq : part2 + a_iq;
        // FP64: old term out, new term in, as the oracle orders them; FP32:
        // the change of r_qi in FP32 (one rounding of a difference far
        // below the row sum), then one FP64 addition.  Empty slots stay 0,
        // and the owner's slot keeps the old r_i until the new one is summed
        const uint64_t upd = null ? 0ull : valid[q] & ~own[q];
        const bool v = __builtin_amdgcn_inverse_ballot_w64(upd);
        if constexpr (sizeof(RT) == 8) {
          const double x = (r[q] - (double)rji[q]) + (double)a_qi;
          r[q] = v ? __builtin_fmax(x, 0.0) : r[q];
        } else {
          const float d = opaque_v(v ? a_qi - rji[q] : 0.0f);
          r[q] = __builtin_fmax(r[q] + (double)d, 0.0);
        }
        m64[q] = !null && __builtin_amdgcn_inverse_ballot_w64(own[q]) ? mnew : m64[q];
      }
    }
    if constexpr (AUX) {
      pcm = cm;
      p_oc = oc;
      p_gi = gi;
      p_mi = mi;
      p_mj = cj.m;
    }
    if (null) part2 = (RT)0;
    scan_rows(K, lane, wave);
    ++e;
    if (__builtin_expect(++rl == rl_end, 0)) {
      if (e >= emax) break;
      draw(lane);
    }
    if (__builtin_expect(!choose(K, lane, wave), 0))
      if (!choose_rare(K, lane, wave)) break;
  }
  if constexpr (AUX) {
    if (pcm.on) comp_store<sizeof(RT) == 8>(A, pcm, lane_cell, p_oc, p_gi, p_mi, p_mj);
  }
  // masses back to HBM (their places are read again rather than held)
  const int tl = wave_cell * 64 + lane_cell;
#pragma unroll
  for (int q = 0; q < KC; ++q) {
    const int K = FIXED ? KC : K_cell, j = tl * K + q;
    if ((FIXED || q < K) && j < n) A.m[A.order[s0 + j]] = m64[q];
  }
  const bool bad_rate = !isfinite(Rtot);
  if (tl == 0) {
    if (bad_rate) atomicOr(&A.state->flags, FLAG_BAD_RATE);
    if (bad_mass) atomicOr(&A.state->flags, FLAG_BAD_MASS);
    const uint32_t n_erode = cnt.n_fast - cnt.n_small - cnt.n_frag;
    const uint32_t n_stick = e - n_null - cnt.n_fast;
    atomicAdd(&A.state->events, (unsigned long long)e);
    if (n_stick) atomicAdd(&A.state->outcomes[OUT_STICK], (unsigned long long)n_stick);
    if (n_erode) atomicAdd(&A.state->outcomes[OUT_ERODE], (unsigned long long)n_erode);
    if (cnt.n_small)
      atomicAdd(&A.state->outcomes[OUT_ERODED_SMALL], (unsigned long long)cnt.n_small);
    if (cnt.n_frag) atomicAdd(&A.state->outcomes[OUT_FRAG], (unsigned long long)cnt.n_frag);
  }
  __builtin_amdgcn_s_setprio(0);
}

template <typename RT, int KMAX, bool FAST, bool PROB, bool AUX, int NW, int LIMIT = kEitherLimit,
          bool BY_K = false>
__device__ __forceinline__ void process_cell(const CollideArgs &A, int cell, char *base, int cap, int wave,
                             int lane, uint32_t step) {
  constexpr int nw = NW;  // waves of the team: 1, or 4 (a compile-time shape per cell body)
  const int s0 = __builtin_amdgcn_readfirstlane(A.cell_start[cell]);
  const int n = __builtin_amdgcn_readfirstlane(A.cell_start[cell + 1]) - s0;
  if (n <= 0) return;
  const int TL = 64 * nw;
  const int K = (n + TL - 1) / TL;
  const RecStore<RT> R(base, cap);
  TeamScratch *const S = (TeamScratch *)(base + (size_t)cap * rec_bytes<RT>());
  const int tl = wave * 64 + lane;
  if (K > KMAX || K * TL > cap) {
    if (tl == 0) atomicOr(&A.state->flags, FLAG_CAPACITY);
    return;
  }
  Gas g;
  {
    // grid sizes opaque per cell: the node lookups' bounds are formed here
    // instead of being held through every cell of a persistent launch
    Model Pl = A.P;
    Pl.grid.nr = opaque_u(Pl.grid.nr);
    Pl.grid.nz = opaque_u(Pl.grid.nz);
    gas_from_primaries(Pl, A.gas + (size_t)cell * 6, g);
  }
  if (!(g.V > 0.0)) {
    if (tl == 0) atomicOr(&A.state->flags, FLAG_BAD_VOLUME);
    return;
  }
  const PairConst<RT> pc = make_pair_const<RT>(A.P, g);

  // ---- members: masses and indices stay in the owning lane's registers ---
  double m64[KMAX];
  int gix[KMAX];
  double ndmax = 0.0;
#pragma unroll
  for (int q = 0; q < KMAX; ++q) {
    const int j = tl * K + q;
    gix[q] = -1;
    m64[q] = 1.0;
    if (q < K && j < n) {
      gix[q] = A.order[s0 + j];
      m64[q] = A.m[gix[q]];
      ndmax = fmax(ndmax, A.M[gix[q]] / (m64[q] * g.V));
    }
  }
  double scale = 1.0;  // FP32 rates are carried as r * scale, a power of two
  if (sizeof(RT) == 4) {
    ndmax = wave_max_nonneg(ndmax);
    if (nw > 1) {
      if (lane == 0) S->tot_i[wave] = ndmax;
      block_lds_sync();
      for (int w = 0; w < nw; ++w) ndmax = fmax(ndmax, S->tot_i[w]);
      block_lds_sync();
    }
    int e2 = 0;
    frexp(ndmax, &e2);
    scale = ldexp(1.0, -e2);
  }
  if (tl == 0) {
    S->gas = g;
    S->cf = make_cellf(A.P, g, scale);
    S->oc = make_outcome_const(A.P);
    // the test kernels have no velocities and never fragment: their zero dv may
    // not reach the mixed form's threshold, also where that is below the range
    // of FP32 (set here, not tested per event: that takes a mixed chain 3%)
    if constexpr (sizeof(RT) == 4 && !FAST)
      if (A.P.kernel != K_PHYSICAL) S->oc.v_frag = INFINITY;
  }
#pragma unroll
  for (int q = 0; q < KMAX; ++q) {
    if (q < K) {
      const bool v = tl * K + q < n;
      R.store(q * TL + tl, v ? make_rec<RT>(A.P, g, m64[q], A.M[gix[q]], scale) : empty_rec<RT>());
    }
  }
  team_sync<NW>();

  // ---- row sums r_i = sum_k r_ik ------------------------------------------
  // The FP32 fast path and FP64, up to four slots per lane, evaluate each
  // unordered pair once (build_rows_pairwise, build_rows_pairwise_team; batched
  // FP64 workload, 250 events: 2.72 against 3.35 ms; own slots one after the
  // other, a quarter of the code: 2.73, its row sums alone 15% slower), but for
  // FP64 teams with few particles (build_rows_plain).  Otherwise partners
  // k = 0..n-1 are read once per group of G own slots and paired with each of
  // them (independent evaluations), and each row adds its terms in canonical
  // order.
  double r[KMAX];
  bool built = false;
  if constexpr ((sizeof(RT) == 8 || FAST) && KMAX == 4) {
    if (nw == 1) {
      build_rows_pairwise<RT, KMAX>(R, pc, K, lane, n, r);
    } else if (sizeof(RT) == 8 && n <= kPlainRows) {
      build_rows_plain<RT, KMAX>(R, pc, tl, n, r);
    } else {
      build_rows_pairwise_team<RT, KMAX>(R, pc, K, wave, lane, n,
                                         (Pair2<RT> *)(base + xbuf_offset<RT>(cap)), r);
    }
    built = true;
  }
  if (!built) {
    constexpr int G = sizeof(RT) == 4 ? 4 : 2;
    static_assert(KMAX % G == 0, "slot groups");
#pragma unroll
    for (int q0 = 0; q0 < KMAX; q0 += G) {
      Rec<RT> mine[G];
      RT acc[G];
#pragma unroll
      for (int g = 0; g < G; ++g) {
        acc[g] = (RT)0;
        if (q0 + g < K) mine[g] = R.load((q0 + g) * TL + tl);
      }
      if (q0 < K) {
        int t2 = 0, q2 = 0;
        for (int k = 0; k < n; ++k) {
          const Rec<RT> rk = R.load(q2 * TL + t2);
#pragma unroll
          for (int g = 0; g < G; ++g) {
            if (q0 + g < K) {
              RT dv, rxy, ryx;
              PairEval<RT, FAST>::run(pc, mine[g], rk, dv, rxy, ryx);
              acc[g] += rxy;
            }
          }
          if (++q2 == K) {
            q2 = 0;
            ++t2;
          }
        }
      }
#pragma unroll
      for (int g = 0; g < G; ++g)
        r[q0 + g] = (q0 + g < K && tl * K + q0 + g < n) ? (double)acc[g] : 0.0;
    }
  }

  if (A.rowsum_dump != nullptr) {
    // test path: the starting row sums as built above, unscaled, at the
    // members' positions in the cell order; no events
#pragma unroll
    for (int q = 0; q < KMAX; ++q)
      if (q < K && tl * K + q < n) A.rowsum_dump[s0 + tl * K + q] = r[q] / scale;
    team_sync<NW>();
    return;
  }

  // ---- events ------------------------------------------------------------
  if constexpr (BY_K) {
    static_assert(KMAX == 4, "one event loop per number of slots");
    switch (K) {
      case 1:
        run_events<RT, 1, true, FAST, PROB, AUX, NW, LIMIT>(A, pc, R, S, cell, s0, n, K, scale, wave,
                                                            lane, step, r, m64);
        break;
      case 2:
        run_events<RT, 2, true, FAST, PROB, AUX, NW, LIMIT>(A, pc, R, S, cell, s0, n, K, scale, wave,
                                                            lane, step, r, m64);
        break;
      case 3:
        run_events<RT, 3, true, FAST, PROB, AUX, NW, LIMIT>(A, pc, R, S, cell, s0, n, K, scale, wave,
                                                            lane, step, r, m64);
        break;
      default:
        run_events<RT, 4, true, FAST, PROB, AUX, NW, LIMIT>(A, pc, R, S, cell, s0, n, K, scale, wave,
                                                            lane, step, r, m64);
    }
  } else {
    run_events<RT, KMAX, false, FAST, PROB, AUX, NW, LIMIT>(A, pc, R, S, cell, s0, n, K, scale, wave,
                                                            lane, step, r, m64);
  }
  team_sync<NW>();  // the region is reused by the next cell
}

// ---------------------------------------------------------------------------
// batched schedule: one persistent launch of four-wave workgroups; big cells
// on four-wave teams (largest first), then small cells on single waves
// (largest first), each wave popping its own work
// ---------------------------------------------------------------------------
//
// Waves per SIMD the mixed form's registers are limited to: three, for the
// throughput of many cells (2500 cells of 64 - 1024 particles, 100 events, test
// kernel: 1208 against 1678 us with two, Maxwell criterion 1811 against 2171); two
// for the time-limited steps that have a kernel of their own without the
// composition mix, where a few cells' chains or the row-sum builds set the pace
// and spills cost more than the third wave gives (first steps of a 5e5 disk: 1.76
// against 1.85 ms for four; one column: 2.71 against 2.77 ms per step; with 8
// fractions, 2e6 particles: 5.45 against 5.15 ms, so not there)
template <typename RT, bool AUX, int LIMIT>
constexpr int waves_per_simd() {
  return sizeof(RT) == 4 && (AUX || LIMIT != kTimeLimited) ? 3 : 2;
}

template <typename RT, int KMAX, bool FAST, bool PROB, bool AUX, int LIMIT = kEitherLimit>
__global__ __launch_bounds__(256, (waves_per_simd<RT, AUX, LIMIT>())) void collide_batched(
    CollideArgs A) {
  extern __shared__ __align__(16) char smem[];
  __shared__ int s_item;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const uint32_t step = A.state->step;
  const size_t small_bytes = region_bytes<RT>(A.small_cap, 1);
  // list lengths from the device plan (zero for a grid that failed validation)
  const int n_big = __builtin_amdgcn_readfirstlane(A.plan->n_big);
  const int n_small = __builtin_amdgcn_readfirstlane(A.plan->n_small);
  int nw = n_big > 0 ? 4 : 1;
  // the first item of a resident launch is given by the workgroup's (one-wave
  // cells: the wave's) place, and the queue begins after those items: all waves
  // at once at one counter take some 10 ns each (2e6 particles with 8 fractions:
  // 4.85 to 4.52 ms a step; first steps of a 5e5 disk, 4: 1.52 to 1.46)
  const int seats = A.seeded ? (int)gridDim.x : 0;
  const int small_seats = nw == 1 ? 4 * seats : 0;  // given out only where no big list comes first
  bool seated = A.seeded != 0;
  for (;;) {
    int cell = -1;
    if (nw == 4) {
      int item = blockIdx.x;
      if (!seated) {
        if (threadIdx.x == 0) s_item = atomicAdd(&A.state->big_head, 1);
        __syncthreads();
        item = __builtin_amdgcn_readfirstlane(s_item) + seats;
        __syncthreads();
      }
      seated = false;
      if (item < n_big)
        cell = __builtin_amdgcn_readfirstlane(A.big_list[item]);
      else
        nw = 1;
    }
    if (nw == 1) {
      int item = wave * (int)gridDim.x + (int)blockIdx.x;
      if (!seated) {
        if (lane == 0) item = atomicAdd(&A.state->small_head, 1);
        item = readlane_i(item, 0) + small_seats;
      }
      seated = false;
      if (item >= n_small) break;
      cell = __builtin_amdgcn_readfirstlane(A.small_list[item]);
    }
    if (nw == 4)
      process_cell<RT, KMAX, FAST, PROB, AUX, 4, LIMIT, KMAX == 4>(A, cell, smem, A.big_cap, wave,
                                                                   lane, step);
    else
      process_cell<RT, KMAX, FAST, PROB, AUX, 1, LIMIT, KMAX == 4>(
          A, cell, smem + (size_t)wave * small_bytes, A.small_cap, 0, lane, step);
  }
}

// plain schedule: one four-wave workgroup per cell, cells in index order
template <typename RT, int KMAX, bool FAST, bool PROB>
__global__ __launch_bounds__(256) void collide_plain(CollideArgs A) {
  extern __shared__ __align__(16) char smem[];
  if (A.plan->bad) return;  // an explicit grid that failed validation
  // the composition mix and the event log are compiled in; they apply when
  // fractions are given or a log is set
  process_cell<RT, KMAX, FAST, PROB, true, 4>(A, blockIdx.x, smem, A.big_cap,
                                              __builtin_amdgcn_readfirstlane(threadIdx.x >> 6),
                                              threadIdx.x & 63, A.state->step);
}

}  // namespace mcd
