// physics.hpp -- gas state, particle state and the pair collision rate of
// the representative-particle method, for device (and host) code.
//
// The paper (arXiv 2507.21239, Summary) fixes the model: a static
// power-law disk, vertically isothermal; representative particles after
// Zsom & Dullemond (2008) colliding inside equal-count cells; relative
// velocities from Brownian motion, turbulence, radial and azimuthal drift and
// settling (the formulas are deferred to Drazkowska et al. 2013).  The forms
// used here: thin-disk gas (Gaussian vertical profile), Epstein / Stokes
// drag switching at a = 9 lambda / 4, Nakagawa-type drift velocities,
// turbulent velocities in the three closed-form regimes of Ormel & Cuzzi
// (2007), the five sources added in quadrature, geometric cross-sections,
// and the swarm rate r_ij = n_j K_ij / max(1, dm_max m_i / m_j).
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace mcd {

// A condition as a lane mask in a general SGPR pair.  A select by VCC has a
// short encoding, and one of those directly after another of the same wave
// takes 23 cycles on gfx950 instead of 5 (measured; three in a row are not
// hidden by three waves per SIMD either); a select by any other pair takes the
// long encoding, which has no such stall.  The empty asm, which clobbers VCC,
// keeps the mask in another pair.
__device__ __forceinline__ uint64_t lane_mask(bool c) {
  uint64_t m = __builtin_amdgcn_ballot_w64(c);
  asm("" : "+s"(m) : : "vcc");
  return m;
}
__device__ __forceinline__ float lane_sel(uint64_t m, float a, float b) {
  return __builtin_amdgcn_inverse_ballot_w64(m) ? a : b;
}

// physical constants, CGS
constexpr double kBoltz = 1.380649e-16;
constexpr double kMassH = 1.6735575e-24;
constexpr double kGrav = 6.67430e-8;
constexpr double kSigmaH2 = 2e-15;
constexpr double kPi = 3.14159265358979323846;
constexpr double kYa = 1.6;  // Ormel & Cuzzi (2007) y*_a

enum : uint32_t {
  DV_BROWNIAN = 1u << 0,
  DV_TURB = 1u << 1,
  DV_RADIAL = 1u << 2,
  DV_AZIMUTHAL = 1u << 3,
  DV_SETTLING = 1u << 4,
  TR_DRIFT = 1u << 8,
  TR_SETTLE = 1u << 9,
  TR_MIX_R = 1u << 10,
  TR_MIX_Z = 1u << 11,
  COAG = 1u << 12,
};
enum { K_PHYSICAL = 0, K_CONSTANT = 1, K_LINEAR = 2 };
enum { OUT_STICK = 0, OUT_ERODE = 1, OUT_ERODED_SMALL = 2, OUT_FRAG = 3 };

// model constants copied to the device by value
// gridded gas on the device: node values on nr radii x nz heights, as
// logarithms (nr == 0: the power-law disk)
struct GasGridView {
  const double *lr;    // [nr] ln r of the radial nodes
  const double *zn;    // [nz] heights of the vertical nodes
  const double *lrho;  // [nr][nz] ln rho_g
  const double *lT;    // [nr][nz] ln T
  const double *lA;    // [nr][nz] ln alpha
  const double *lS;    // [nr] ln Sigma_g
  int32_t nr, nz;
};

struct Model {
  double sigma_g0, T0, p, q, alpha, v_frag, erosion_ratio, rho_s, mu, m_star, r_ref;
  double dm_max, erosion_chi, r_in, r_col, k0, m0, frag_width;
  uint32_t flags;
  int32_t kernel, column, n_comp, frag_mode;
  uint32_t key0, key1;
  GasGridView grid;
};

enum : int32_t { FRAG_SHARP = 0, FRAG_RAMP = 1, FRAG_MAXWELL = 2 };

// the model parameters a collision outcome reads, gathered per cell into the
// team's LDS scratch: read there once per event instead of being held (and
// spilled) in scalar registers for the whole persistent launch
struct alignas(16) OutcomeConst {
  double v_frag, erosion_ratio, erosion_chi, m0, dm_max, frag_width;
  int32_t kernel, frag_mode, n_comp, pad;
};

__host__ __device__ inline OutcomeConst make_outcome_const(const Model &P) {
  OutcomeConst o;
  o.v_frag = P.v_frag;
  o.erosion_ratio = P.erosion_ratio;
  o.erosion_chi = P.erosion_chi;
  o.m0 = P.m0;
  o.dm_max = P.dm_max;
  o.frag_width = P.frag_width;
  o.kernel = P.kernel;
  o.frag_mode = P.frag_mode;
  o.n_comp = P.n_comp;
  o.pad = 0;
  return o;
}

struct DiskPoint {
  double Sigma_g, T, cs, Omega, H, rho_g;
};

// x^-e: the half-integer exponents of disk models (1/2, 1, 3/2) by roots and
// products in place of pow, whose 300 FP64 instructions set the pace of a kernel
// over all particles.  The root and the product are each corrected by their
// residue, so that the result is as near as one rounding brings it (0.501 ulp at
// most over 2e6 arguments on the host; uncorrected 1.5 for 1/2 and 2.4 for 3/2, a
// microsecond less per 1e6 particles; the host's pow 0.51).  The cells' gas keeps
// pow: a last bit there could round a cell's FP32 constants the other way.
__host__ __device__ inline double inverse_power(double x, double e) {
  if (e == 1.0) return 1.0 / x;
  if ((e == 0.5 || e == 1.5) && x > 1e-90 && x < 1e90) {
    const double s = 1.0 / sqrt(x), s2 = s * s;
    // what s lacks: (1 - s^2 x) s / 2, the low half of s^2 included
    const double c = 0.5 * s * fma(-fma(s, s, -s2), x, fma(-s2, x, 1.0));
    if (e == 0.5) return s + c;
    const double t = s * s2;  // (s + c) / x, corrected by its residue over x
    return fma(fma(-t, x, s) + c, s2, t);
  }
  return pow(x, -e);
}

template <bool ROOTS = false>
__host__ __device__ inline DiskPoint disk_at(const Model &P, double r, double z) {
  DiskPoint d;
  const double x = r / P.r_ref;
  d.Sigma_g = P.sigma_g0 * (ROOTS ? inverse_power(x, P.p) : pow(x, -P.p));
  d.T = P.T0 * (ROOTS ? inverse_power(x, P.q) : pow(x, -P.q));
  d.cs = sqrt(kBoltz * d.T / (P.mu * kMassH));
  d.Omega = sqrt(kGrav * P.m_star / (r * r * r));
  d.H = d.cs / d.Omega;
  d.rho_g = d.Sigma_g / (sqrt(2.0 * kPi) * d.H) * exp(-(z * z) / (2.0 * d.H * d.H));
  return d;
}

// gas at one point: density, temperature, turbulence, sound speed, Kepler
// frequency, scale height, pressure slope s = -d ln P / d ln r (eta v_K =
// c_s^2 s / (2 Omega r)) and the radial-diffusion correction factor c (the
// random walk drifts by D c / r: the logarithmic r-derivative of
// r Sigma_g D with D ~ alpha c_s H, the drift under which an axisymmetric
// random walk keeps a tracer distributed like the gas)
struct LocalGas {
  double rho_g, T, alpha, cs, Omega, H, slopeP, corr;
};

// cell of a node array containing x, clamped to the first / last cell, and
// the fractional position in it (0 or 1 outside the nodes)
__host__ __device__ inline void grid_locate(const double *nodes, int n, double x, int &k,
                                            double &w) {
  if (!(x > nodes[0])) {
    k = 0;
    w = 0.0;
    return;
  }
  if (!(x < nodes[n - 1])) {
    k = n - 2;
    w = 1.0;
    return;
  }
  int lo = 0, hi = n - 1;  // nodes[lo] <= x < nodes[hi]
  while (hi - lo > 1) {
    const int mid = lo + (hi - lo) / 2;
    if (x < nodes[mid])
      hi = mid;
    else
      lo = mid;
  }
  k = lo;
  w = (x - nodes[lo]) / (nodes[lo + 1] - nodes[lo]);
}

// power-law disk, or the gridded gas: bilinear in (ln r, z) of ln rho_g,
// ln T and ln alpha, with the r-slopes of those interpolants at this height;
// the surface density's slope from its radial nodes
template <bool ROOTS = false>
__host__ __device__ inline LocalGas local_gas_at(const Model &P, double r, double z) {
  LocalGas o;
  const GasGridView &G = P.grid;
  if (G.nr == 0) {
    const DiskPoint d = disk_at<ROOTS>(P, r, z);
    o.rho_g = d.rho_g;
    o.T = d.T;
    o.cs = d.cs;
    o.Omega = d.Omega;
    o.H = d.H;
    o.alpha = P.alpha;
    o.slopeP = P.p + (P.q + 3.0) / 2.0;
    o.corr = 2.5 - P.q - P.p;  // Sigma_g ~ r^-p, c_s H ~ r^(3/2 - q), times r
    return o;
  }
  int k, l;
  double wx, wz;
  grid_locate(G.lr, G.nr, log(r), k, wx);
  grid_locate(G.zn, G.nz, z, l, wz);
  const int64_t i00 = (int64_t)k * G.nz + l, i10 = i00 + G.nz, i01 = i00 + 1, i11 = i10 + 1;
  const double dx = G.lr[k + 1] - G.lr[k];
  const double *f[3] = {G.lrho, G.lT, G.lA};
  double val[3], slope[3];
  for (int q = 0; q < 3; ++q) {
    const double *a = f[q];
    val[q] = (1.0 - wx) * (1.0 - wz) * a[i00] + wx * (1.0 - wz) * a[i10] +
             (1.0 - wx) * wz * a[i01] + wx * wz * a[i11];
    slope[q] = ((1.0 - wz) * (a[i10] - a[i00]) + wz * (a[i11] - a[i01])) / dx;
  }
  o.rho_g = exp(val[0]);
  o.T = exp(val[1]);
  o.alpha = exp(val[2]);
  o.cs = sqrt(kBoltz * o.T / (P.mu * kMassH));
  o.Omega = sqrt(kGrav * P.m_star / (r * r * r));
  o.H = o.cs / o.Omega;
  o.slopeP = -(slope[0] + slope[1]);  // pressure rho_g c_s^2 ~ rho_g T
  const double dlnS = (G.lS[k + 1] - G.lS[k]) / dx;
  o.corr = dlnS + slope[2] + slope[1] + 2.5;  // alpha T r^(3/2), times r
  return o;
}

// gas state of a cell, from its six primaries (V, rho_g, T, alpha, r_c,
// zeta = z_c / H)
struct Gas {
  double V, rho_g, T, alpha, r_c, zeta;
  double cs, Omega, H, z_c, eta_vK, v_th, lambda, nu, Re, St_eta, Vg2;
};

__host__ __device__ inline void gas_from_primaries(const Model &P, const double *prim, Gas &g) {
  g.V = prim[0];
  g.rho_g = prim[1];
  g.T = prim[2];
  g.alpha = prim[3];
  g.r_c = prim[4];
  g.zeta = prim[5];
  g.cs = sqrt(kBoltz * g.T / (P.mu * kMassH));
  g.Omega = sqrt(kGrav * P.m_star / (g.r_c * g.r_c * g.r_c));
  g.H = g.cs / g.Omega;
  g.z_c = g.zeta * g.H;
  // midplane pressure-gradient velocity: P ~ r^-(p + (q+3)/2)
  g.eta_vK = 0.5 * (g.cs * g.cs) / (g.Omega * g.r_c) *
             (P.grid.nr ? local_gas_at(P, g.r_c, g.z_c).slopeP : (P.p + (P.q + 3.0) / 2.0));
  g.v_th = sqrt(8.0 / kPi) * g.cs;
  g.lambda = P.mu * kMassH / (g.rho_g * kSigmaH2);
  g.nu = 0.5 * g.v_th * g.lambda;
  g.Re = g.alpha * g.cs * g.H / g.nu;
  g.St_eta = 1.0 / sqrt(g.Re);
  g.Vg2 = 1.5 * g.alpha * g.cs * g.cs;
}

// power-law disk at (r, z): Sigma_g, T, c_s, Omega, H, rho_g
__host__ __device__ inline double stopping_time(double rho_s, double a, double rho_g, double v_th,
                                                double lambda, double nu) {
  if (a < 2.25 * lambda) return rho_s * a / (rho_g * v_th);  // Epstein
  return 2.0 * rho_s * a * a / (9.0 * nu * rho_g);           // Stokes
}

// per-particle record used by the pair rate, in the rate precision RT
template <typename RT>
struct Rec {
  RT m;    // mass
  RT im;   // 1/m
  RT a;    // radius
  RT St;   // Stokes number
  RT h;    // St^2 / (St + St_eta)
  RT q1;   // 1 / (1 + St)
  RT vr;   // radial drift velocity
  RT vp;   // azimuthal velocity relative to Keplerian
  RT vz;   // settling velocity at the cell height
  RT nd;   // swarm number density M/(m V), times the cell's rate scale
  RT ist;  // 1 / St
  RT Mn;   // swarm mass M / V times the rate scale (nd = Mn / m)
};

// the FP32 record carries sqrt(pi) a in place of a, so that the collision
// cross-section pi (a_i + a_j)^2 needs no extra product
constexpr double kSqrtPi = 1.7724538509055160273;
template <typename RT>
__host__ __device__ constexpr double radius_factor() {
  return sizeof(RT) == 4 ? kSqrtPi : 1.0;
}

// Stokes numbers and their regime line St_eta as the FP64 pair rates hold them:
// in a vacuum both are infinite, and the rates have to find the regime of large
// Stokes numbers and divide there (NaN stays NaN)
constexpr double kStMax = 0x1p1022, kStEtaMax = 0x1p1021;
__host__ __device__ inline double at_most(double x, double top) { return x > top ? top : x; }

// particle state in FP64 (the precompute is always FP64), rounded to RT
template <typename RT>
__host__ __device__ inline Rec<RT> make_rec(const Model &P, const Gas &g, double m, double M,
                                            double nd_scale) {
  const double a = cbrt(3.0 * m / (4.0 * kPi * P.rho_s));
  const double ts = stopping_time(P.rho_s, a, g.rho_g, g.v_th, g.lambda, g.nu);
  const double St = ts * g.Omega;
  Rec<RT> o;
  o.m = (RT)m;
  o.im = (RT)(1.0 / m);
  o.a = (RT)(a * radius_factor<RT>());
  o.St = (RT)at_most(St, kStMax);
  o.ist = (RT)(1.0 / St);
  o.h = (RT)(St * St / (St + g.St_eta));
  o.q1 = (RT)(1.0 / (1.0 + St));
  o.vr = (RT)(-2.0 * g.eta_vK * St / (1.0 + St * St));
  o.vp = (RT)(-g.eta_vK / (1.0 + St * St));
  o.vz = (RT)(-g.z_c * g.Omega * St / (1.0 + St));
  o.nd = (RT)(M / (m * g.V) * nd_scale);
  o.Mn = (RT)(M * (nd_scale / g.V));
  return o;
}

// per-cell constants of the FP32 particle state (mixed precision): the
// same formulas as make_rec with the cell factors folded in single precision
struct alignas(16) CellF {
  float ca;     // 3 / (4 pi rho_s)
  float a_sw;   // Epstein / Stokes switch radius 9 lambda / 4
  float tE;     // Epstein stopping time per unit radius rho_s / (rho_g v_th)
  float tS;     // Stokes stopping time per unit radius^2 2 rho_s / (9 nu rho_g)
  float Om, Ste, m2eta, meta, mzO;
  float pad;
  double nd_fac;  // rate scale / V
};

__host__ __device__ inline CellF make_cellf(const Model &P, const Gas &g, double scale) {
  CellF c;
  c.ca = (float)(3.0 / (4.0 * kPi * P.rho_s));
  c.a_sw = (float)(2.25 * g.lambda);
  c.tE = (float)(P.rho_s / (g.rho_g * g.v_th));
  c.tS = (float)(2.0 * P.rho_s / (9.0 * g.nu * g.rho_g));
  c.Om = (float)g.Omega;
  c.Ste = (float)g.St_eta;
  c.m2eta = (float)(-2.0 * g.eta_vK);
  c.meta = (float)(-g.eta_vK);
  c.mzO = (float)(-g.z_c * g.Omega);
  c.pad = 0.0f;
  c.nd_fac = scale / g.V;
  return c;
}

// per-cell constants of the pair rate
template <typename RT>
struct PairConst {
  RT cBM;      // 8 k T / pi
  RT Vg2;      // large-eddy velocity squared
  RT St_eta;   // Kolmogorov Stokes number Re^-1/2
  RT dm_max;
  RT inv_dm;   // 1 / dm_max (infinite when grouping is off)
  RT k0;
  uint32_t flags;
  int32_t kernel;
};

template <typename RT>
__host__ __device__ inline PairConst<RT> make_pair_const(const Model &P, const Gas &g) {
  PairConst<RT> c;
  c.cBM = (RT)(8.0 * kBoltz * g.T / kPi);
  c.Vg2 = (RT)g.Vg2;
  c.St_eta = (RT)at_most(g.St_eta, kStEtaMax);
  c.dm_max = (RT)P.dm_max;
  c.inv_dm = P.dm_max > 0.0 ? (RT)(1.0 / P.dm_max) : (RT)INFINITY;
  c.k0 = (RT)P.k0;
  c.flags = P.flags;
  c.kernel = P.kernel;
  return c;
}

// FP32 particle state of the mixed path (after a collision changed m)
// Mn: the particle's swarm mass times the cell's density factor, as the
// record holds it ((float)(M * nd_fac))
__device__ inline Rec<float> make_rec_f(const CellF &c, double m, float Mn) {
  const float mf = (float)m;
  const float a = cbrtf(mf * c.ca);
  const float ts = a < c.a_sw ? c.tE * a : c.tS * a * a;
  const float St = ts * c.Om;
  const float q1 = __builtin_amdgcn_rcpf(1.0f + St);
  const float w = __builtin_amdgcn_rcpf(1.0f + St * St);
  Rec<float> r;
  r.m = mf;
  r.im = __builtin_amdgcn_rcpf(mf);
  r.a = a * (float)kSqrtPi;
  r.St = St;
  r.ist = __builtin_amdgcn_rcpf(St);
  r.h = St * St * __builtin_amdgcn_rcpf(St + c.Ste);
  r.q1 = q1;
  r.vr = c.m2eta * St * w;
  r.vp = c.meta * w;
  r.vz = c.mzO * St * q1;
  r.nd = Mn * r.im;
  r.Mn = Mn;
  return r;
}

// precision-specific square root and the FP32 division: FP64 correctly rounded;
// FP32 through the hardware reciprocal and square root (about 1 ulp)
__device__ inline float pdiv(float a, float b) { return a * __builtin_amdgcn_rcpf(b); }
__device__ inline double psqrt(double x) { return sqrt(x); }
__device__ inline float psqrt(float x) { return __builtin_amdgcn_sqrtf(x); }

// turbulent relative velocity squared (Ormel & Cuzzi 2007 closed forms)
template <typename RT>
__device__ inline RT dv2_turb(const PairConst<RT> &c, const Rec<RT> &x, const Rec<RT> &y) {
  const bool xb = x.St > y.St;
  const RT St1 = xb ? x.St : y.St, St2 = xb ? y.St : x.St;
  // FP64: the three regimes over one division, chosen before it, instead of
  // up to three divisions in branches that a wave's pairs take one after the
  // other (batched FP64 workload: 4.31 to 3.35 ms, with the grouping factor
  // below).  h grows with St, so |h_x - h_y| is h_1 - h_2.  Large Stokes numbers
  // take numerator and denominator times 2^-1000, which changes no bit of an
  // ordinary quotient and keeps the product of thin gas's numbers in range
  // (2.65 to 2.67 ms)
  if constexpr (sizeof(RT) == 8) {
    const bool tiny = St1 < c.St_eta, inter = !tiny && St1 < 1.0;
    const double sum = St1 + St2, q = kYa * St1 + St2;
    const double cubic = 2.0 * ((1.0 / (1.0 + kYa)) * (St1 * St1) * q + St2 * St2 * St2);
    constexpr double k = 0x1p-1000;
    const double num = tiny ? (St1 - St2) * fabs(x.h - y.h) : inter ? cubic : fma(sum, k, 2.0 * k);
    const double den = tiny ? sum : inter ? sum * q : fma(St1, k, k) * (1.0 + St2);
    const double rest = inter ? (2.0 * kYa - 1.0) * St1 - St2 : 0.0;
    return c.Vg2 * (rest + num / den);
  } else {
    if (St1 < c.St_eta) {
      const float h1 = xb ? x.h : y.h, h2 = xb ? y.h : x.h;
      return pdiv(c.Vg2 * (St1 - St2), St1 + St2) * (h1 - h2);
    }
    if (St1 < 1.0f) {
      const float eps = pdiv(St2, St1);
      const float br = (float)(2.0 * kYa) - (1.0f + eps) +
                       pdiv(2.0f, 1.0f + eps) *
                           ((float)(1.0 / (1.0 + kYa)) + pdiv(eps * eps * eps, (float)kYa + eps));
      return c.Vg2 * St1 * br;
    }
    return c.Vg2 * (x.q1 + y.q1);
  }
}

// relative velocity of the pair (five sources in quadrature)
template <typename RT>
__device__ inline RT rel_velocity(const PairConst<RT> &c, const Rec<RT> &x, const Rec<RT> &y) {
  RT dv2 = (RT)0;
  if (c.flags & DV_BROWNIAN) dv2 += c.cBM * (x.im + y.im);
  if (c.flags & DV_TURB) dv2 += dv2_turb(c, x, y);
  if (c.flags & DV_RADIAL) {
    const RT d = x.vr - y.vr;
    dv2 += d * d;
  }
  if (c.flags & DV_AZIMUTHAL) {
    const RT d = x.vp - y.vp;
    dv2 += d * d;
  }
  if (c.flags & DV_SETTLING) {
    const RT d = x.vz - y.vz;
    dv2 += d * d;
  }
  return psqrt(dv2);
}

// symmetric collision kernel K_xy; dv receives the relative velocity
template <typename RT>
__device__ inline RT pair_kernel(const PairConst<RT> &c, const Rec<RT> &x, const Rec<RT> &y,
                                 RT &dv) {
  if (c.kernel == K_CONSTANT) {
    dv = (RT)0;
    return c.k0;
  }
  if (c.kernel == K_LINEAR) {
    dv = (RT)0;
    return c.k0 * (x.m + y.m);
  }
  dv = rel_velocity(c, x, y);
  const RT s = x.a + y.a;
  if (sizeof(RT) == 4) return s * s * dv;  // the FP32 radii carry sqrt(pi)
  return (RT)kPi * s * s * dv;
}

// FP32 rates of a pair for the physical kernel with all five velocity
// sources: r_xy = n_y K_xy / max(1, dm m_x/m_y) and r_yx, and the relative
// velocity.  Same quantities as rel_velocity / pair_kernel / swarm_rate,
// arranged for few instructions: the Ormel & Cuzzi regimes evaluated
// branch-free from eps = St2/St1 with one shared reciprocal of
// (1 + eps)(y_a + eps) -- (St1 - St2)/(St1 + St2) = (1 - eps)/(1 + eps) and
// 2/(1 + eps) (1/(1 + y_a) + eps^3/(y_a + eps)) =
// 2 ((y_a + eps)/(1 + y_a) + eps^3) / ((1 + eps)(y_a + eps)) --, fused
// multiply-adds for the quadrature sum, sqrt(pi) folded into the radii.
//
// BRANCH (the row-sum build): the grouping factors behind a (uniform) test of
// dm_max, which ends the block of every pair; the build's blocks of up to 16
// pairs run faster so (row sums of 4096 cells of 64 - 1024 particles: 679
// against 759 us), the events' straight code without it (the batched workload:
// 10.9 against 11.6 ms).
template <bool BRANCH = false>
__device__ inline void pair_rates_all(const PairConst<float> &c, const Rec<float> &x,
                                      const Rec<float> &y, float &dv, float &rxy, float &ryx) {
  constexpr float ya = (float)kYa;
  constexpr float c1 = (float)(1.0 / (1.0 + kYa));
  constexpr float b0 = (float)(2.0 * kYa - 1.0);
  // h and q1 in registers before the arithmetic: otherwise their loads are
  // deferred into the regime choice, a second wait on LDS per pair
  if constexpr (BRANCH) asm volatile("" ::"v"(x.h), "v"(x.q1), "v"(y.h), "v"(y.q1));
  float dv2 = c.cBM * (x.im + y.im);
  // selects: by masks in the build's dense pairs (row sums of the cells above:
  // 627 against 671 us), left to the compiler in the events' chain, where the
  // masks' longer path costs what the stall does
  const bool xb = x.St > y.St;
  uint64_t xm = 0;
  if constexpr (BRANCH) xm = lane_mask(xb);
  auto sel = [&](float a, float b) __attribute__((always_inline)) {
    if constexpr (BRANCH) return lane_sel(xm, a, b);
    return xb ? a : b;
  };
  const float St1 = sel(x.St, y.St);
  const float ist1 = sel(x.ist, y.ist);
  // h = St^2 / (St + St_eta) grows with St: the larger-St particle has the larger h
  const float hd = fabsf(x.h - y.h);
  const float eps = sel(y.St, x.St) * ist1;
  const float ye = ya + eps;
  const float rd = __builtin_amdgcn_rcpf((1.0f + eps) * ye);
  const float tiny = (1.0f - eps) * (ye * rd) * hd;
  const float inter = St1 * (b0 - eps + 2.0f * rd * fmaf(ye, c1, eps * eps * eps));
  const float heavy = x.q1 + y.q1;
  // the regime is chosen by selects, not branches: the two candidate values
  // pass through an empty asm so that the optimizer cannot sink their
  // arithmetic into per-regime blocks (which serialise a wave's pairs)
  float tn = tiny, it = inter;
  asm("" : "+v"(tn), "+v"(it));
  float turb;
  if constexpr (BRANCH)
    turb = lane_sel(lane_mask(St1 < c.St_eta), tn, lane_sel(lane_mask(St1 < 1.0f), it, heavy));
  else
    turb = St1 < c.St_eta ? tn : (St1 < 1.0f ? it : heavy);
  dv2 = fmaf(c.Vg2, turb, dv2);
  float d = x.vr - y.vr;
  dv2 = fmaf(d, d, dv2);
  d = x.vp - y.vp;
  dv2 = fmaf(d, d, dv2);
  d = x.vz - y.vz;
  dv2 = fmaf(d, d, dv2);
  dv = __builtin_amdgcn_sqrtf(dv2);
  const float s = x.a + y.a;
  const float K = s * s * dv;
  rxy = y.nd * K;
  ryx = x.nd * K;
  // min(1, m_y / (dm_max m_x)): 1 with grouping off, where inv_dm is infinite
  if (!BRANCH || c.dm_max > 0.0f) {
    rxy *= fminf(1.0f, y.m * (x.im * c.inv_dm));
    ryx *= fminf(1.0f, x.m * (y.im * c.inv_dm));
  }
}

// rates of representative particle x against swarm y and the other way round
// given K_xy: n_y K / max(1, dm_max m_x / m_y).  FP64: n_y K min(1, m_y /
// (dm_max m_x)); as dm_max is at most 1, only the heavier particle's factor
// can be below one, so a pair takes one division
__device__ inline void swarm_rates(const PairConst<double> &c, const Rec<double> &x,
                                   const Rec<double> &y, double K, double &rxy, double &ryx) {
  rxy = y.nd * K;
  ryx = x.nd * K;
  if (c.dm_max > 0.0) {
    const bool xh = x.m > y.m;
    const double hi = xh ? x.m : y.m, lo = xh ? y.m : x.m;
    const double f = fmin(1.0, lo / (c.dm_max * hi));
    rxy *= xh ? f : 1.0;
    ryx *= xh ? 1.0 : f;
  }
}
// FP32: the same factor as n_y K min(1, m_y / (dm_max m_x)), no reciprocal
__device__ inline float swarm_rate(const PairConst<float> &c, const Rec<float> &x,
                                   const Rec<float> &y, float K) {
  float r = y.nd * K;
  if (c.dm_max > 0.0f) r *= fminf(1.0f, y.m * (x.im * c.inv_dm));
  return r;
}
__device__ inline void swarm_rates(const PairConst<float> &c, const Rec<float> &x,
                                   const Rec<float> &y, float K, float &rxy, float &ryx) {
  rxy = swarm_rate(c, x, y, K);
  ryx = swarm_rate(c, y, x, K);
}

// fragment mass: inverse-CDF draw from the mass-weighted distribution
// ~ m^(-5/6) (number slope 11/6) on [lo, hi]
__host__ __device__ inline double frag_draw(double lo, double hi, double u) {
  if (!(hi > lo)) return lo;
  const double slo = sqrt(cbrt(lo)), shi = sqrt(cbrt(hi));
  const double x = slo + u * (shi - slo);
  const double x2 = x * x;
  return x2 * x2 * x2;
}

// probability that a collision at mean relative velocity dv fragments (or
// erodes): linear ramp from (1 - w) v_frag to v_frag, or the tail above
// v_frag of the Maxwell speed distribution with mean dv (scale a =
// dv sqrt(pi/8)): erfc(x) + 2/sqrt(pi) x exp(-x^2), x = v_frag / (sqrt(2) a)
// in the precision T of dv (double for the FP64 form, float for the mixed one)
template <typename PP, typename T>
__host__ __device__ inline T frag_probability(const PP &P, T dv) {
  const T vf = (T)P.v_frag;
  if (P.frag_mode == FRAG_RAMP) {
    const T lo = ((T)1 - (T)P.frag_width) * vf;
    if (dv <= lo) return (T)0;
    if (dv >= vf) return (T)1;
    return (dv - lo) / (vf - lo);
  }
  if (P.frag_mode == FRAG_MAXWELL) {
    if (!(dv > (T)0)) return (T)0;
    const T x = (T)2 * vf / (sqrt((T)kPi) * dv);
    return erfc(x) + (T)2 / sqrt((T)kPi) * x * exp(-x * x);
  }
  return dv < vf ? (T)0 : (T)1;
}

// grouping factor max(1, dm_max m_i / m_j)
__host__ __device__ inline double group_factor(double dm_max, double mi, double mj) {
  if (!(dm_max > 0.0)) return 1.0;
  const double g = dm_max * mi / mj;
  return g < 1.0 ? 1.0 : g;
}

// collision outcome for representative particle i (mass mi) hitting a body
// of swarm j (mass mj) at relative velocity dv, in the FP64 form; returns the
// outcome code (the mixed form's rules: event_outcome)
template <typename PP>
__host__ __device__ inline int outcome(const PP &P, bool fast, double mi, double mj, double u,
                                       double &m_new) {
  // grouped mass grp * mj; the eroded mass chi grp mj
  const double grp = group_factor(P.dm_max, mi, mj);
  const double gm = grp * mj, em = P.erosion_chi * grp * mj;
  if (P.kernel != K_PHYSICAL || !fast) {
    m_new = mi + gm;
    return OUT_STICK;
  }
  const double big = mi > mj ? mi : mj;
  const double small = mi > mj ? mj : mi;
  if (big / small >= P.erosion_ratio) {
    if (mi >= mj) {
      const double m = mi - em;
      m_new = m > P.m0 ? m : P.m0;
      return OUT_ERODE;
    }
    m_new = frag_draw(P.m0, mi, u);
    return OUT_ERODED_SMALL;
  }
  m_new = frag_draw(P.m0, big, u);
  return OUT_FRAG;
}

}  // namespace mcd
