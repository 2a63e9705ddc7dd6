// binning.hip -- equal-count adaptive grid (paper, Summary: every cell holds
// the same number of representative particles).
//
// Radial zones: active particles ranked by (r, index), zone k holds ranks
// [floor(k Na / n_r), floor((k+1) Na / n_r)).  Cells: inside a zone, ranked
// by (z, index) and split the same way into n_z cells.
//
// Rank by r: one reduction gives the active count and the range of the IEEE
// bit patterns of r (non-negative doubles order like their bits); a 32-bit
// key (bits - min) >> shift, with shift chosen so keys keep 31 bits, is
// sorted by a stable least-significant-digit radix sort (8-bit digits, tiles
// of 2048 keys per 256-thread workgroup, per-tile digit histograms, a scan
// over tiles per digit, and a scatter that first orders the tile by digit in
// LDS and then writes each digit's run contiguously).  Stability keeps equal
// keys in index order; a fix-up pass then orders each run of equal keys by
// the full 64-bit pattern and index, so the result is the exact (r, index)
// order.  Rank by z: each zone is a contiguous range of the r order; one
// workgroup loads its members' (z bits, index) pairs and sorts them with a
// bitonic network held in registers.  Zones larger than that sort takes
// (8192) go the global path: 64-bit radix sort by z, then a stable radix pass
// by zone.
#include <algorithm>

#include "device_common.hpp"
#include "internal.hpp"

namespace mcd {

constexpr int kRadixThreads = 256;
constexpr int kRadixItems = 8;
constexpr int kRadixTile = kRadixThreads * kRadixItems;

int radix_tiles(int64_t n) {
  return (int)std::max<int64_t>(1, (n + kRadixTile - 1) / kRadixTile);
}

__device__ inline uint64_t key_bits(double x) {
  return (uint64_t)__double_as_longlong(x + 0.0);  // -0 -> +0
}

// ---------------------------------------------------------------------------
// active count and range of the r bit patterns
// ---------------------------------------------------------------------------
// per-workgroup partials {min, max, count}, which every workgroup of the next
// kernel combines for itself (no atomics: a few thousand 64-bit atomics on one
// address serialise; and no launch of 4 us for 256 values)
__device__ inline void minmax_wave(uint64_t &lo, uint64_t &hi, uint64_t &cnt) {
  for (int off = 32; off > 0; off >>= 1) {
    const uint64_t l2 = __shfl_xor(lo, off, 64), h2 = __shfl_xor(hi, off, 64);
    lo = l2 < lo ? l2 : lo;
    hi = h2 > hi ? h2 : hi;
    cnt += __shfl_xor(cnt, off, 64);
  }
}

__device__ inline void minmax_block(uint64_t &lo, uint64_t &hi, uint64_t &cnt) {
  __shared__ uint64_t s[3][16];
  minmax_wave(lo, hi, cnt);
  const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    s[0][w] = lo;
    s[1][w] = hi;
    s[2][w] = cnt;
  }
  __syncthreads();
  lo = ~0ull;
  hi = 0ull;
  cnt = 0ull;
  for (int k = 0; k < nw; ++k) {
    lo = s[0][k] < lo ? s[0][k] : lo;
    hi = s[1][k] > hi ? s[1][k] : hi;
    cnt += s[2][k];
  }
}

__global__ __launch_bounds__(1024) void k_minmax_part(const double *__restrict__ r,
                                                     const uint8_t *__restrict__ active,
                                                     int64_t N, uint64_t *part) {
  uint64_t lo = ~0ull, hi = 0ull, cnt = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N;
       i += (int64_t)gridDim.x * blockDim.x) {
    if (active[i]) {
      const uint64_t b = key_bits(r[i]);
      lo = b < lo ? b : lo;
      hi = b > hi ? b : hi;
      ++cnt;
    }
  }
  minmax_block(lo, hi, cnt);
  if (threadIdx.x == 0) {
    part[3 * blockIdx.x] = lo;
    part[3 * blockIdx.x + 1] = hi;
    part[3 * blockIdx.x + 2] = cnt;
  }
}

// the workgroup's (256 threads) view of the partials
__device__ inline BinState combine_parts(const uint64_t *__restrict__ part, int n_part) {
  static_assert(kMinmaxParts <= 256, "one partial per thread");
  const int k = threadIdx.x;
  uint64_t lo = ~0ull, hi = 0ull, cnt = 0;
  if (k < n_part) {
    lo = part[3 * k];
    hi = part[3 * k + 1];
    cnt = part[3 * k + 2];
  }
  minmax_block(lo, hi, cnt);
  return BinState{lo, hi, (uint32_t)cnt, 0u};
}

__device__ inline int key_shift(const BinState &bs) {
  const uint64_t span = bs.max_bits - bs.min_bits;
  const int bits = span ? 64 - __builtin_clzll(span) : 0;
  return bits > 31 ? bits - 31 : 0;
}

// 32-bit keys of one radix tile, and the tile's histogram of the first
// digit (the first pass needs no histogram kernel of its own).  The first
// workgroup leaves the active count and readies the state for the collision
// launch and the end of the step
__global__ __launch_bounds__(256) void k_keys_r32_hist(const double *__restrict__ r,
                                                       const uint8_t *__restrict__ active, int64_t N,
                                                       const uint64_t *part, int n_part,
                                                       DevState *st, uint32_t *keys,
                                                       int32_t *vals, uint32_t *hist, int tiles) {
  __shared__ uint32_t h[256];
  h[threadIdx.x] = 0u;
  const BinState bs = combine_parts(part, n_part);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->n_active = (int32_t)bs.count;
    st->big_head = 0;
    st->small_head = 0;
    st->bin_step = st->step;
  }
  const int sh = key_shift(bs);
  const uint64_t lo = bs.min_bits;
  const int64_t base = (int64_t)blockIdx.x * kRadixTile;
#pragma unroll
  for (int it = 0; it < kRadixItems; ++it) {
    const int64_t i = base + it * kRadixThreads + threadIdx.x;
    if (i < N) {
      const uint32_t k = active[i] ? (uint32_t)((key_bits(r[i]) - lo) >> sh) : 0xFFFFFFFFu;
      keys[i] = k;
      vals[i] = (int32_t)i;
      atomicAdd(&h[k & 255u], 1u);
    }
  }
  __syncthreads();
  hist[(size_t)threadIdx.x * tiles + blockIdx.x] = h[threadIdx.x];
}

__global__ __launch_bounds__(256) void k_keys_from_double(const double *__restrict__ x,
                                                          const uint8_t *__restrict__ active,
                                                          int64_t N, uint64_t *keys, int32_t *vals) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  keys[i] = active[i] ? key_bits(x[i]) : ~0ull;
  vals[i] = (int32_t)i;
}

// ---------------------------------------------------------------------------
// stable LSD radix pass, 8-bit digits
// ---------------------------------------------------------------------------
template <typename KeyT>
__global__ __launch_bounds__(256) void k_radix_hist(const KeyT *__restrict__ keys, int64_t N,
                                                    int shift, uint32_t *hist, int tiles) {
  __shared__ uint32_t h[256];
  h[threadIdx.x] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * kRadixTile;
#pragma unroll
  for (int it = 0; it < kRadixItems; ++it) {
    const int64_t i = base + it * kRadixThreads + threadIdx.x;
    if (i < N) atomicAdd(&h[(uint32_t)(keys[i] >> shift) & 255u], 1u);
  }
  __syncthreads();
  hist[(size_t)threadIdx.x * tiles + blockIdx.x] = h[threadIdx.x];
}

// inclusive prefix sum over the wave
__device__ inline uint32_t wave_incl_scan_u32(uint32_t v) {
  int x = (int)v;
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);  // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);  // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true);  // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true);  // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, true);  // row_bcast:15 into rows 1, 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, true);  // row_bcast:31 into rows 2, 3
  return (uint32_t)x;
}

// two inclusive prefix sums over the 256 threads of a workgroup, one barrier
__device__ inline void block_incl_scan2(uint32_t &a, uint32_t &b, uint32_t (*s)[2]) {
  const int wave = threadIdx.x >> 6;
  a = wave_incl_scan_u32(a);
  b = wave_incl_scan_u32(b);
  if ((threadIdx.x & 63) == 63) {
    s[wave][0] = a;
    s[wave][1] = b;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < 3; ++w) {
    a += w < wave ? s[w][0] : 0u;
    b += w < wave ? s[w][1] : 0u;
  }
}

// exclusive scan of one digit's row of tile counts; row total -> digit_tot
__global__ __launch_bounds__(256) void k_radix_scan_rows(uint32_t *hist, int tiles,
                                                         uint32_t *digit_tot) {
  __shared__ uint32_t s[4][2];
  uint32_t *row = hist + (size_t)blockIdx.x * tiles;
  const int per = (tiles + 255) / 256;
  const int start = threadIdx.x * per;
  uint32_t loc = 0;
  for (int k = 0; k < per; ++k) {
    const int x = start + k;
    if (x < tiles) loc += row[x];
  }
  uint32_t inc = loc, none = 0u;
  block_incl_scan2(inc, none, s);
  uint32_t run = inc - loc;
  for (int k = 0; k < per; ++k) {
    const int x = start + k;
    if (x < tiles) {
      const uint32_t c = row[x];
      row[x] = run;
      run += c;
    }
  }
  if (threadIdx.x == 255) digit_tot[blockIdx.x] = inc;
}

// Stable scatter of one tile.  Element order within the tile is (wave, item,
// lane): a wave owns a quarter of the tile, finds the earlier lanes of an item
// with the same digit by eight ballots and chains its items through digit
// counters of its own, so that the tile takes four barriers.  The tile is then
// written to LDS in digit order, and each digit's run is copied to its global
// range, so consecutive lanes write consecutive words.  Bound by the passes
// over keys and indices and the launch: at 1e6 particles 9.5 us a pass of 32-bit
// keys, 13.5 with the items of all four waves in turn and five barriers each.
// TWICE: the indices go to vcopy as well.
template <typename KeyT, bool TWICE>
__global__ __launch_bounds__(256) void k_radix_scatter(const KeyT *__restrict__ kin,
                                                       const int32_t *__restrict__ vin,
                                                       KeyT *__restrict__ kout,
                                                       int32_t *__restrict__ vout,
                                                       int32_t *__restrict__ vcopy, int64_t N,
                                                       int shift, const uint32_t *hist,
                                                       const uint32_t *digit_tot, int tiles) {
  __shared__ KeyT sk[kRadixTile];
  __shared__ int32_t sv[kRadixTile];
  __shared__ uint32_t gofs[256];     // global less local position of digit d
  __shared__ uint32_t wcnt[4][256];  // count, then first local position, of digit d by wave
  __shared__ uint32_t s[4][2];
  constexpr int kWaveItems = kRadixItems * 64;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int64_t tbase = (int64_t)blockIdx.x * kRadixTile;
  const int tile_n = (int)std::min<int64_t>(kRadixTile, N - tbase);

  KeyT key[kRadixItems];
  int32_t val[kRadixItems];
#pragma unroll
  for (int it = 0; it < kRadixItems; ++it) {
    const int li = wave * kWaveItems + it * 64 + lane;
    key[it] = li < tile_n ? kin[tbase + li] : (KeyT)0;
    val[it] = li < tile_n ? vin[tbase + li] : 0;
  }
  const uint32_t gtot = digit_tot[tid], gtile = hist[(size_t)tid * tiles + blockIdx.x];
#pragma unroll
  for (int w = 0; w < 4; ++w) wcnt[w][tid] = 0u;
  __syncthreads();
  const uint64_t lt_mask = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  uint32_t pos[kRadixItems];  // rank among the wave's elements of the digit
#pragma unroll
  for (int it = 0; it < kRadixItems; ++it) {
    const bool valid = wave * kWaveItems + it * 64 + lane < tile_n;
    const uint32_t digit = (uint32_t)(key[it] >> shift) & 255u;
    uint64_t same = ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const bool bit = (digit >> b) & 1u;
      const uint64_t bb = ballot(bit);
      same &= bit ? bb : ~bb;
    }
    const uint32_t rank = (uint32_t)__popcll(same & lt_mask);
    const uint32_t before = wcnt[wave][digit];
    wave_lds_sync();
    if (valid && rank == 0) wcnt[wave][digit] = before + (uint32_t)__popcll(same);
    wave_lds_sync();
    pos[it] = before + rank;
  }
  __syncthreads();
  {
    uint32_t c[4], cnt = 0u;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      c[w] = wcnt[w][tid];
      cnt += c[w];
    }
    uint32_t inc = cnt, ginc = gtot;
    block_incl_scan2(inc, ginc, s);
    uint32_t run = inc - cnt;
    gofs[tid] = (ginc - gtot) + gtile - run;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      wcnt[w][tid] = run;
      run += c[w];
    }
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < kRadixItems; ++it) {
    if (wave * kWaveItems + it * 64 + lane < tile_n) {
      const uint32_t p = wcnt[wave][(uint32_t)(key[it] >> shift) & 255u] + pos[it];
      sk[p] = key[it];
      sv[p] = val[it];
    }
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < kRadixItems; ++it) {
    const int p = it * kRadixThreads + tid;
    if (p < tile_n) {
      const KeyT k = sk[p];
      const uint32_t g = gofs[(uint32_t)(k >> shift) & 255u] + (uint32_t)p;
      kout[g] = k;
      vout[g] = sv[p];
      if (TWICE) vcopy[g] = sv[p];
    }
  }
}

// have_hist: the tile histograms of this pass are already in hist; vcopy: where
// a second copy of the indices goes, or nullptr
template <typename KeyT>
static hipError_t radix_pass(KeyT *const keys[2], int32_t *const vals[2], uint32_t *hist,
                             uint32_t *digit_tot, int &cur, int64_t N, int shift, hipStream_t s,
                             bool have_hist = false, int32_t *vcopy = nullptr) {
  const int tiles = radix_tiles(N);
  if (!have_hist) k_radix_hist<KeyT><<<tiles, kRadixThreads, 0, s>>>(keys[cur], N, shift, hist, tiles);
  k_radix_scan_rows<<<256, 256, 0, s>>>(hist, tiles, digit_tot);
  auto scatter = vcopy ? k_radix_scatter<KeyT, true> : k_radix_scatter<KeyT, false>;
  scatter<<<tiles, kRadixThreads, 0, s>>>(keys[cur], vals[cur], keys[cur ^ 1], vals[cur ^ 1], vcopy,
                                          N, shift, hist, digit_tot, tiles);
  cur ^= 1;
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// exact order inside runs of equal 32-bit keys: by full r bits, then index.
// Stability leaves every run in index order, so a run needs work only if two
// neighbours in it differ in r.  The first such position of each run
// insertion-sorts the run in by_r, a copy of the order, by (bits of r, index);
// keys and vals are read-only here.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_fix_ties(const uint32_t *__restrict__ keys,
                                                  const int32_t *__restrict__ vals,
                                                  const double *__restrict__ r, const DevState *st,
                                                  int32_t *by_r) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t na = st->n_active;
  if (p + 1 >= na) return;
  const uint32_t k = keys[p];
  if (keys[p + 1] != k) return;
  auto differs = [&](int64_t a) {  // from its successor, of the same key
    return key_bits(r[vals[a]]) != key_bits(r[vals[a + 1]]);
  };
  if (!differs(p)) return;
  int64_t s = p;
  while (s > 0 && keys[s - 1] == k) {
    if (differs(s - 1)) return;  // an earlier position of this run does the work
    --s;
  }
  int64_t e = p + 2;
  while (e < na && keys[e] == k) ++e;
  for (int64_t a = s + 1; a < e; ++a) {
    const int32_t v = by_r[a];
    const uint64_t bv = key_bits(r[v]);
    int64_t b = a - 1;
    while (b >= s) {
      const int32_t u = by_r[b];
      const uint64_t bu = key_bits(r[u]);
      if (bu < bv || (bu == bv && u < v)) break;
      by_r[b + 1] = u;
      --b;
    }
    by_r[b + 1] = v;
  }
}

__global__ __launch_bounds__(256) void k_copy_i32(const int32_t *__restrict__ a,
                                                  int32_t *__restrict__ b, int64_t N) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < N) b[i] = a[i];
}

// zone of the particle of rank p: the largest k with floor(k Na / n_r) <= p
__global__ __launch_bounds__(256) void k_zone(const int32_t *__restrict__ by_r, int64_t N, int n_r,
                                              const DevState *st, int32_t *zone) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= N) return;
  const int64_t na = st->n_active;
  zone[by_r[p]] = p < na ? (int32_t)(((p + 1) * (int64_t)n_r - 1) / na) : n_r;
}

__global__ __launch_bounds__(256) void k_keys_zone(const int32_t *__restrict__ vals,
                                                   const int32_t *__restrict__ zone, int64_t N,
                                                   uint64_t *keys) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < N) keys[i] = (uint64_t)(uint32_t)zone[vals[i]];
}

// ---------------------------------------------------------------------------
// order of each zone by (z, index): one workgroup per zone runs a bitonic
// network over the zone padded to P = 8 x threads (a power of two, >= 512).
// An element is 32 bits: its z bit pattern, range-reduced over the zone
// ((bits - min) >> shift) to the bits that are left (19 at the largest P), above
// its position in the r order, so that an exchange is one minimum and one
// maximum.  Thread t keeps positions 8t .. 8t+7 in registers: strides below 8
// compare inside a thread, strides 8 .. 256 pair lanes of one wave (no
// barrier), strides of 512 and up exchange through LDS between barriers.
// Each run of equal reduced keys is then sorted by (full bits, index), so the
// result is the exact (z, index) order.  Runs are a few elements long unless
// the zone's z nearly coincide; a zone with a run of more than kZoneRun takes
// the network over 64-bit elements (32 bits of z above the index) instead.
// Bound by the network's instructions and the gather of z: 1e6 particles in 500
// zones take 29 us, 59 with 64-bit elements throughout; with all heights equal,
// where both networks run, 62 against 56.
// ---------------------------------------------------------------------------
constexpr int kZoneItems = 8;
constexpr int kZoneRun = 16;

// the element at position p takes the smaller of (own, partner) if it is the
// lower position of an ascending pair or the upper one of a descending pair
__device__ inline void keep_one(uint64_t &k, uint64_t k2, int p, int stride, int size) {
  const bool want_min = ((p & stride) == 0) == ((p & size) == 0);
  const bool take = want_min ? k > k2 : k2 > k;
  k = take ? k2 : k;
}

// value of lane (lane ^ LM) of the wave.  Lane xors below 16 are DPP moves
// (VALU): quad permutes give xor 1 and xor 2; a half-row mirror (xor 7)
// followed by a quad reverse (xor 3) gives xor 4; a row mirror (xor 15)
// followed by a half-row mirror gives xor 8.  Xors 16 and 32 use the LDS
// permute network.
template <int LM>
__device__ inline uint32_t lane_xor(uint32_t v) {
  const int x = (int)v;
  if constexpr (LM == 1) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, x, 0xB1, 0xf, 0xf, true);
  } else if constexpr (LM == 2) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, x, 0x4E, 0xf, 0xf, true);
  } else if constexpr (LM == 4) {
    const int y = __builtin_amdgcn_update_dpp(0, x, 0x141, 0xf, 0xf, true);
    return (uint32_t)__builtin_amdgcn_update_dpp(0, y, 0x1B, 0xf, 0xf, true);
  } else if constexpr (LM == 8) {
    const int y = __builtin_amdgcn_update_dpp(0, x, 0x140, 0xf, 0xf, true);
    return (uint32_t)__builtin_amdgcn_update_dpp(0, y, 0x141, 0xf, 0xf, true);
  } else {
    return (uint32_t)__shfl_xor(x, LM, 64);
  }
}

// one exchange phase between lanes (strides 8 .. 256): for these strides the
// bits tested by the pair direction lie above the thread's own 8 positions
template <int LM>
__device__ inline void zone_lane_phase(uint64_t (&key)[kZoneItems], int base, int stride,
                                       int size) {
  const bool want_min = ((base & stride) == 0) == ((base & size) == 0);
#pragma unroll
  for (int e = 0; e < kZoneItems; ++e) {
    const uint32_t lo = lane_xor<LM>((uint32_t)key[e]);
    const uint32_t hi = lane_xor<LM>((uint32_t)(key[e] >> 32));
    const uint64_t k2 = ((uint64_t)hi << 32) | lo;
    const bool take = want_min ? key[e] > k2 : k2 > key[e];
    key[e] = take ? k2 : key[e];
  }
}

template <int S>
__device__ inline void zone_reg_phase(uint64_t (&key)[kZoneItems], int base, int size) {
#pragma unroll
  for (int e = 0; e < kZoneItems; ++e) {
    if (e & S) continue;
    const bool up = ((base + e) & size) == 0;
    if ((key[e] > key[e + S]) == up) {
      const uint64_t t = key[e];
      key[e] = key[e + S];
      key[e + S] = t;
    }
  }
}

// the network over 64-bit elements: reduced z above the index, one comparison;
// with shift > 0 the runs of equal reduced z are sorted again by (full bits,
// index).  lk, lz: LDS of P elements each
__device__ void zone_sort_wide(const uint64_t (&bits)[kZoneItems], const int32_t (&idx)[kZoneItems],
                               uint64_t zmin, uint64_t range, int nk, int P,
                               const double *__restrict__ z, uint64_t *lk, uint64_t *lz,
                               int32_t *__restrict__ order) {
  const int base = threadIdx.x * kZoneItems;
  const int shift = (range >> 32) ? 32 - __clzll((long long)range) : 0;
  uint64_t key[kZoneItems];
#pragma unroll
  for (int e = 0; e < kZoneItems; ++e)
    key[e] = base + e < nk ? (((bits[e] - zmin) >> shift) << 32) | (uint32_t)idx[e] : ~0ull;
  for (int size = 2; size <= P; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      if (stride >= 64 * kZoneItems) {
#pragma unroll
        for (int e = 0; e < kZoneItems; ++e) lk[base + e] = key[e];
        __syncthreads();
#pragma unroll
        for (int e = 0; e < kZoneItems; ++e) keep_one(key[e], lk[(base + e) ^ stride], base + e, stride, size);
        __syncthreads();
      } else if (stride >= kZoneItems) {
        switch (stride / kZoneItems) {
          case 1: zone_lane_phase<1>(key, base, stride, size); break;
          case 2: zone_lane_phase<2>(key, base, stride, size); break;
          case 4: zone_lane_phase<4>(key, base, stride, size); break;
          case 8: zone_lane_phase<8>(key, base, stride, size); break;
          case 16: zone_lane_phase<16>(key, base, stride, size); break;
          default: zone_lane_phase<32>(key, base, stride, size); break;
        }
      } else if (stride == 4) {
        zone_reg_phase<4>(key, base, size);
      } else if (stride == 2) {
        zone_reg_phase<2>(key, base, size);
      } else {
        zone_reg_phase<1>(key, base, size);
      }
    }
  }
  if (shift > 0) {
    // runs of equal reduced keys, re-sorted by (full bits, index) by the
    // thread that holds the run's first position.  Only members of such runs
    // need their full bits (read again from z): a reduced key keeps 32
    // significant bits of the zone's range, so runs are rare
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kZoneItems; ++e) lk[base + e] = key[e];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kZoneItems; ++e) {
      const int p = base + e;
      if (p >= nk) continue;
      const uint32_t h = (uint32_t)(lk[p] >> 32);
      const bool tied = (p + 1 < nk && (uint32_t)(lk[p + 1] >> 32) == h) ||
                        (p > 0 && (uint32_t)(lk[p - 1] >> 32) == h);
      if (tied) lz[p] = key_bits(z[(int32_t)(uint32_t)key[e]]);
    }
    __syncthreads();
    for (int e = 0; e < kZoneItems; ++e) {
      const int p = base + e;
      const uint32_t h = (uint32_t)(lk[p] >> 32);
      if (p + 1 >= nk || (uint32_t)(lk[p + 1] >> 32) != h) continue;
      if (p > 0 && (uint32_t)(lk[p - 1] >> 32) == h) continue;
      int end = p + 2;
      while (end < nk && (uint32_t)(lk[end] >> 32) == h) ++end;
      for (int a = p + 1; a < end; ++a) {  // insertion sort of [p, end)
        const uint64_t kv = lk[a], zv = lz[a];
        const uint32_t iv = (uint32_t)kv;
        int b = a - 1;
        while (b >= p && (lz[b] > zv || (lz[b] == zv && (uint32_t)lk[b] > iv))) {
          lk[b + 1] = lk[b];
          lz[b + 1] = lz[b];
          --b;
        }
        lk[b + 1] = kv;
        lz[b + 1] = zv;
      }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kZoneItems; ++e) key[e] = lk[base + e];
  }
#pragma unroll
  for (int e = 0; e < kZoneItems; ++e)
    if (base + e < nk) order[base + e] = (int32_t)(uint32_t)key[e];
}

// 32-bit exchanges: between lanes (xor LM), and inside a thread (stride S);
// selects by masks, see lane_mask
__device__ __forceinline__ uint32_t mask_sel(uint64_t m, uint32_t a, uint32_t b) {
  return __builtin_amdgcn_inverse_ballot_w64(m) ? a : b;
}
template <int LM>
__device__ __forceinline__ void lane_phase32(uint32_t (&key)[kZoneItems], uint64_t want_min) {
#pragma unroll
  for (int e = 0; e < kZoneItems; ++e) {
    uint32_t a = key[e], b;
    if constexpr (LM >= 16) {
      // both results together hold the own and the partner's value
      if constexpr (LM == 16) {
        const auto v = __builtin_amdgcn_permlane16_swap(a, a, false, false);
        a = v[0], b = v[1];
      } else {
        const auto v = __builtin_amdgcn_permlane32_swap(a, a, false, false);
        a = v[0], b = v[1];
      }
    } else {
      b = lane_xor<LM>(a);
    }
    key[e] = mask_sel(want_min, min(a, b), max(a, b));
  }
}
template <int S>
__device__ __forceinline__ void reg_phase32(uint32_t (&key)[kZoneItems], uint64_t up) {
#pragma unroll
  for (int e = 0; e < kZoneItems; ++e) {
    if (e & S) continue;
    const uint32_t a = min(key[e], key[e + S]), b = max(key[e], key[e + S]);
    key[e] = mask_sel(up, a, b);
    key[e + S] = mask_sel(up, b, a);
  }
}
// (the first sizes: directions known at compile time)
template <int S, int SIZE>
__device__ __forceinline__ void first_phase32(uint32_t (&key)[kZoneItems]) {
#pragma unroll
  for (int e = 0; e < kZoneItems; ++e) {
    if (e & S) continue;
    const uint32_t a = min(key[e], key[e + S]), b = max(key[e], key[e + S]);
    key[e] = (e & SIZE) ? b : a;
    key[e + S] = (e & SIZE) ? a : b;
  }
}

__global__ __launch_bounds__(1024) void k_zone_sort(const int32_t *__restrict__ by_r,
                                                    const double *__restrict__ z, int n_r,
                                                    const DevState *st, int32_t *order) {
  extern __shared__ __align__(16) char smem[];
  __shared__ uint64_t s_lo[16], s_hi[16];
  __shared__ int s_long;
  const int64_t na = st->n_active;
  const int zk = blockIdx.x;
  const int64_t b0 = (int64_t)zk * na / n_r, b1 = (int64_t)(zk + 1) * na / n_r;
  const int nk = (int)(b1 - b0);
  if (nk <= 0) return;
  const int P = blockDim.x * kZoneItems, pos_bits = 31 - __clz(P);
  const int tid = threadIdx.x;
  const int base = tid * kZoneItems;
  uint64_t *lz = (uint64_t *)smem;         // full bits, in r order
  int32_t *li = (int32_t *)(lz + P);       // index, in r order
  uint32_t *lk = (uint32_t *)(li + P);     // elements
  uint64_t bits[kZoneItems];
  int32_t idx[kZoneItems];
  uint64_t lo = ~0ull, hi = 0ull;
#pragma unroll
  for (int e = 0; e < kZoneItems; ++e) {
    // any thread may take any position: the network sorts them all.  Lanes
    // read consecutive words here
    const int p = e * (int)blockDim.x + tid;
    idx[e] = 0x7FFFFFFF;
    bits[e] = 0;
    if (p < nk) idx[e] = by_r[b0 + p];
  }
#pragma unroll
  for (int e = 0; e < kZoneItems; ++e) {
    const int p = e * (int)blockDim.x + tid;
    if (p < nk) {
      bits[e] = key_bits(z[idx[e]]);
      lo = bits[e] < lo ? bits[e] : lo;
      hi = bits[e] > hi ? bits[e] : hi;
      lz[p] = bits[e];
      li[p] = idx[e];
    }
  }
  // range of the zone's bit patterns
  uint64_t none = 0;
  minmax_wave(lo, hi, none);
  if ((tid & 63) == 0) {
    s_lo[tid >> 6] = lo;
    s_hi[tid >> 6] = hi;
  }
  if (tid == 0) s_long = 0;
  __syncthreads();
  for (int w = 0; w < (int)blockDim.x >> 6; ++w) {
    lo = s_lo[w] < lo ? s_lo[w] : lo;
    hi = s_hi[w] > hi ? s_hi[w] : hi;
  }
  const uint64_t range = hi - lo;
  const int used = range ? 64 - __clzll((long long)range) : 0;
  const int shift = max(0, used - (32 - pos_bits));
  uint32_t key[kZoneItems];
#pragma unroll
  for (int e = 0; e < kZoneItems; ++e) {
    const int p = e * (int)blockDim.x + tid;
    key[e] = p < nk ? ((uint32_t)((bits[e] - lo) >> shift) << pos_bits) | (uint32_t)p : ~0u;
  }
  first_phase32<1, 2>(key);
  first_phase32<2, 4>(key);
  first_phase32<1, 4>(key);
  for (int size = 8; size <= P; size <<= 1) {
    const uint64_t up = lane_mask((base & size) == 0);
    for (int stride = size >> 1; stride >= kZoneItems; stride >>= 1) {
      const uint64_t want_min = lane_mask((base & stride) != 0) ^ up;
      if (stride >= 64 * kZoneItems) {
        uint4 *own = (uint4 *)(lk + base);
        own[0] = make_uint4(key[0], key[1], key[2], key[3]);
        own[1] = make_uint4(key[4], key[5], key[6], key[7]);
        __syncthreads();
        const uint4 *other = (const uint4 *)(lk + (base ^ stride));
        const uint4 a = other[0], b = other[1];
        const uint32_t k2[kZoneItems] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
        for (int e = 0; e < kZoneItems; ++e)
          key[e] = mask_sel(want_min, min(key[e], k2[e]), max(key[e], k2[e]));
        __syncthreads();
      } else {
        switch (stride / kZoneItems) {
          case 1: lane_phase32<1>(key, want_min); break;
          case 2: lane_phase32<2>(key, want_min); break;
          case 4: lane_phase32<4>(key, want_min); break;
          case 8: lane_phase32<8>(key, want_min); break;
          case 16: lane_phase32<16>(key, want_min); break;
          default: lane_phase32<32>(key, want_min); break;
        }
      }
    }
    reg_phase32<4>(key, up);
    reg_phase32<2>(key, up);
    reg_phase32<1>(key, up);
  }
  {
    uint4 *own = (uint4 *)(lk + base);
    own[0] = make_uint4(key[0], key[1], key[2], key[3]);
    own[1] = make_uint4(key[4], key[5], key[6], key[7]);
  }
  __syncthreads();
  // runs of equal reduced keys (the elements past nk belong to none)
  const uint32_t pmask = (uint32_t)P - 1u;
#pragma unroll
  for (int e = 0; e < kZoneItems; ++e) {
    const int p = base + e;
    if (p + kZoneRun < nk && (lk[p + kZoneRun] >> pos_bits) == (key[e] >> pos_bits)) s_long = 1;
  }
  __syncthreads();
  if (s_long) {
#pragma unroll
    for (int e = 0; e < kZoneItems; ++e) {
      const int p = base + e;
      idx[e] = p < nk ? li[p] : 0x7FFFFFFF;
      bits[e] = p < nk ? lz[p] : 0;
    }
    __syncthreads();
    zone_sort_wide(bits, idx, lo, range, nk, P, z, lz, lz + P, order + b0);
    return;
  }
  for (int e = 0; e < kZoneItems; ++e) {
    const int p = base + e;
    const uint32_t h = key[e] >> pos_bits;
    if (p + 1 >= nk || (lk[p + 1] >> pos_bits) != h) continue;
    if (p > 0 && (lk[p - 1] >> pos_bits) == h) continue;
    int end = p + 2;
    while (end < nk && (lk[end] >> pos_bits) == h) ++end;
    for (int a = p + 1; a < end; ++a) {  // insertion sort of [p, end)
      const uint32_t kv = lk[a];
      const uint64_t zv = lz[kv & pmask];
      const int32_t iv = li[kv & pmask];
      int b = a - 1;
      while (b >= p) {
        const uint64_t zb = lz[lk[b] & pmask];
        if (!(zb > zv || (zb == zv && li[lk[b] & pmask] > iv))) break;
        lk[b + 1] = lk[b];
        --b;
      }
      lk[b + 1] = kv;
    }
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < kZoneItems; ++e) {
    const int p = e * (int)blockDim.x + tid;
    if (p < nk) order[b0 + p] = li[lk[p] & pmask];
  }
}

// member ranges, edges, volumes and gas primaries of every cell
__global__ __launch_bounds__(256) void k_cells(Model P, int n_r, int n_z,
                                               const double *__restrict__ r,
                                               const double *__restrict__ z,
                                               const int32_t *__restrict__ by_r,
                                               const int32_t *__restrict__ order,
                                               const DevState *st, int32_t *cell_start,
                                               double *geom, double *gas) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  const int nc = n_r * n_z;
  if (c >= nc) return;
  const int64_t na = st->n_active;
  const int k = c / n_z, l = c % n_z;
  const int64_t b0 = (int64_t)k * na / n_r, b1 = (int64_t)(k + 1) * na / n_r;
  const int64_t nk = b1 - b0;
  const int64_t s0 = b0 + (int64_t)l * nk / n_z, s1 = b0 + (int64_t)(l + 1) * nk / n_z;
  cell_start[c] = (int32_t)s0;
  if (c == nc - 1) cell_start[nc] = (int32_t)na;
  double r_lo = 0.0, r_hi = 0.0, z_lo = 0.0, z_hi = 0.0;
  if (nk > 0) {
    r_lo = b0 == 0 ? r[by_r[b0]] : 0.5 * (r[by_r[b0 - 1]] + r[by_r[b0]]);
    r_hi = b1 == na ? r[by_r[b1 - 1]] : 0.5 * (r[by_r[b1 - 1]] + r[by_r[b1]]);
  }
  if (s1 > s0) {
    z_lo = s0 == b0 ? 0.0 : 0.5 * (z[order[s0 - 1]] + z[order[s0]]);
    z_hi = s1 == b1 ? z[order[s1 - 1]] : 0.5 * (z[order[s1 - 1]] + z[order[s1]]);
  }
  const double r_c = P.column ? P.r_col : 0.5 * (r_lo + r_hi);
  const double z_c = 0.5 * (z_lo + z_hi);
  const double V = P.column ? 2.0 * (z_hi - z_lo)
                            : 2.0 * kPi * (r_hi * r_hi - r_lo * r_lo) * (z_hi - z_lo);
  double *gm = geom + (size_t)c * 5;
  gm[0] = r_lo;
  gm[1] = r_hi;
  gm[2] = z_lo;
  gm[3] = z_hi;
  gm[4] = V;
  double *gs = gas + (size_t)c * 6;
  if (s1 > s0) {
    const LocalGas d = local_gas_at(P, r_c, z_c);
    gs[0] = V;
    gs[1] = d.rho_g;
    gs[2] = d.T;
    gs[3] = d.alpha;
    gs[4] = r_c;
    gs[5] = z_c / d.H;
  } else {
    for (int f = 0; f < 6; ++f) gs[f] = 0.0;
  }
}

// padded size of the zone sort: a power of two, at least 512 (one full wave)
int zone_sort_size(int64_t zone_max) {
  int P = 64 * kZoneItems;
  while (P < zone_max) P <<= 1;
  return P;
}

hipError_t launch_binning(const Model &P, int n_r, int n_z, const double *r, const double *z,
                          const uint8_t *active, int64_t N, BinBuffers &b, int32_t *cell_start,
                          int32_t *order, double *geom, double *gas, DevState *state,
                          hipStream_t s) {
  if (N <= 0 || N > b.cap) return hipErrorInvalidValue;
  const unsigned g1 = (unsigned)((N + 255) / 256);
  hipError_t e;
  // 1. rank by (r, index)
  const unsigned n_part = (unsigned)std::min<int64_t>((N + 1023) / 1024, kMinmaxParts);
  k_minmax_part<<<n_part, 1024, 0, s>>>(r, active, N, b.part);
  const int tiles = radix_tiles(N);
  k_keys_r32_hist<<<tiles, kRadixThreads, 0, s>>>(r, active, N, b.part, (int)n_part, state,
                                                  b.k32[0], b.vals[0], b.hist, tiles);
  int cur = 0;
  for (int sh = 0; sh < 32; sh += 8)
    if ((e = radix_pass<uint32_t>(b.k32, b.vals, b.hist, b.digit_tot, cur, N, sh, s, sh == 0,
                                  sh == 24 ? b.by_r : nullptr)) != hipSuccess)
      return e;
  k_fix_ties<<<g1, 256, 0, s>>>(b.k32[cur], b.vals[cur], r, state, b.by_r);
  // 2. rank by (z, index) inside each zone
  const int64_t zone_max = (N + n_r - 1) / n_r;  // no zone holds more
  if (zone_max > kZoneSortMax && (b.keys[0] == nullptr || b.zone == nullptr))
    return hipErrorInvalidValue;  // the workspace holds no buffers of the global path
  if (zone_max <= kZoneSortMax) {
    const int Pz = zone_sort_size(zone_max);
    const size_t lds = (size_t)Pz * 2 * sizeof(uint64_t);  // keys, then full bits for the runs
    if (lds > 64 * 1024) {
      e = hipFuncSetAttribute((const void *)k_zone_sort, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)lds);
      if (e != hipSuccess) return e;
    }
    k_zone_sort<<<n_r, Pz / kZoneItems, lds, s>>>(b.by_r, z, n_r, state, order);
  } else {
    k_zone<<<g1, 256, 0, s>>>(b.by_r, N, n_r, state, b.zone);
    cur = 0;
    k_keys_from_double<<<g1, 256, 0, s>>>(z, active, N, b.keys[0], b.vals[0]);
    for (int sh = 0; sh < 64; sh += 8)
      if ((e = radix_pass<uint64_t>(b.keys, b.vals, b.hist, b.digit_tot, cur, N, sh, s)) != hipSuccess)
        return e;
    if (n_r > 1) {
      k_keys_zone<<<g1, 256, 0, s>>>(b.vals[cur], b.zone, N, b.keys[cur]);
      for (int sh = 0; sh < 16 && (n_r >> sh) > 0; sh += 8)
        if ((e = radix_pass<uint64_t>(b.keys, b.vals, b.hist, b.digit_tot, cur, N, sh, s)) != hipSuccess)
          return e;
    }
    k_copy_i32<<<g1, 256, 0, s>>>(b.vals[cur], order, N);
  }
  // 3. cells
  const int nc = n_r * n_z;
  k_cells<<<(nc + 255) / 256, 256, 0, s>>>(P, n_r, n_z, r, z, b.by_r, order, state, cell_start,
                                           geom, gas);
  return hipGetLastError();
}

}  // namespace mcd
