// physics.h -- per-cell and per-interface arithmetic of the FISH sweeps,
// as device functions for gfx950.  Templated on the storage/arithmetic type T
// (double, or float with FP64 pressure recovery) and on the sweep axis D so
// that every component index is a compile-time constant (no scratch).
//
// FP32 arithmetic uses the hardware reciprocal and square root (1 ulp) in
// place of the IEEE division/square-root sequences; FP64 arithmetic refines
// the hardware estimates by Newton (reciprocal) and Goldschmidt (square root)
// steps, without the IEEE sequences' range scaling and special-case fixups,
// and divides by multiplying with the reciprocal.
//
// Sect. 2.1-2.4 of the FISH paper; equation numbers are the printed ones.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

// Multiply-adds are fused only within one source expression (never across
// statements), so the rounding of every value is fixed by the source alone:
// the kernels that stream the same arithmetic in different layouts (lanes,
// pairs of positions, strided pencils, any work shape) give bitwise the same
// result.
#pragma clang fp contract(on)

namespace fish {

enum { RHO = 0, MX = 1, MY = 2, MZ = 3, EN = 4 };

__device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float fsqrt(float x) { return __builtin_amdgcn_sqrtf(x); }

// 1/x in FP64: the hardware estimate (relative error about 5e-8) and two
// Newton steps r <- r + r (1 - x r), each squaring the relative error.  Equal
// to the IEEE quotient on every sampled x whose reciprocal is a finite
// nonzero number; 0, infinite x and an overflowing reciprocal give NaN (the
// sweeps take reciprocals of densities, cell widths and sums of same-signed
// slopes, which are positive and finite in any valid state).
__device__ __forceinline__ double rcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = fma(-x, r, 1.0);
  r = fma(r, e, r);
  e = fma(-x, r, 1.0);
  return fma(r, e, r);
}

// sqrt(x) in FP64: Goldschmidt's iteration from the hardware estimate y of
// 1/sqrt(x), carrying s -> sqrt(x) and h -> 1/(2 sqrt(x)) (s = x y, h = y/2),
// one coupled step and two residual corrections s += h (x - s^2).  Within one
// ulp of the IEEE root for positive finite x, subnormals included (equal on
// nearly every sample); sqrt(0) = 0, negative x gives NaN, +inf gives NaN
// (IEEE: inf), so a non-finite or negative argument still leaves a
// non-finite result.
__device__ __forceinline__ double fsqrt(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  double s = x * y, h = 0.5 * y;
  const double e = fma(-h, s, 0.5);
  s = fma(s, e, s);
  h = fma(h, e, h);
  double d = fma(-s, s, x);
  s = fma(d, h, s);
  d = fma(-s, s, x);
  s = fma(d, h, s);
  return x == 0.0 ? x : s;
}

// 1/rho in FP64 for the pressure recovery: the FP64 reciprocal above in FP64
// mode (the same value as the sweep's 1/rho); in FP32 mode the hardware
// FP32 reciprocal refined by one Newton step in FP64 (relative error ~1e-14,
// far below the FP32 storage rounding of E).
__device__ __forceinline__ double rinv64(double rho, double) { return rcp(rho); }
__device__ __forceinline__ double rinv64(double rho, float rho32) {
  const double r0 = (double)__builtin_amdgcn_rcpf(rho32);
  return r0 * (2.0 - rho * r0);
}

// max(x, 0) that keeps a NaN (the result of an invalid operation has its sign
// bit clear): one integer instruction on the sign.  In FP64 only the high word
// is tested, so a negative x leaves a subnormal >= 0 in place of zero.
__device__ __forceinline__ float nonneg(float x) { return __int_as_float(max(__float_as_int(x), 0)); }
__device__ __forceinline__ double nonneg(double x) {
  const long long b = __double_as_longlong(x);
  return __longlong_as_double(((long long)max((int)(b >> 32), 0) << 32) | (b & 0xffffffffll));
}

// max(a, b) of two speeds >= 0.  FP32: the bit patterns of non-negative numbers
// are ordered as the numbers, NaNs above all, so a NaN in either operand wins.
// FP64: a NaN in b wins, one in a gives b (the compare of the bit patterns costs
// 0.4% of a step).  A cell is the right one (b) of its left interface, so a cell
// without a speed makes its state bad in both.
__device__ __forceinline__ float speed_max(float a, float b) {
  return __int_as_float(max(__float_as_uint(a), __float_as_uint(b)));
}
__device__ __forceinline__ double speed_max(double a, double b) { return a > b ? a : b; }

// A cell's centred field and b^2 (in FP64, for the pressure).  The field is
// fixed during L_d, so the half-step state takes both over from the first
// evaluation of the cell.
template <typename T>
struct FieldQ {
  T b[3];
  double b2;
};
template <typename T>
__device__ __forceinline__ FieldQ<T> field_quantities(const T* b) {
  FieldQ<T> f;
#pragma unroll
  for (int k = 0; k < 3; ++k) f.b[k] = b[k];
  const double bx = (double)b[0], by = (double)b[1], bz = (double)b[2];
  f.b2 = bx * bx + by * by + bz * bz;
  return f;
}

// Quantities of one cell for a sweep along D (Sect. 2.2), the flux and the
// speeds as the halves that Eqs. (24)-(34) take of them: F is half the flux of
// Eq. (17) with x replaced by D, but for the mass flux (half_flux), d half the
// freezing speed |v_D| + c_F of Eq. (21), vd and cF half its terms.  cF, cS and xiE
// (= -(E + p), the energy entry of Eq. 50) only for HSE.
//
// A half velocity makes them for a few products a cell, where halving what the
// interfaces form takes 35 a position; the scalings are exact, so the results
// are the same.  Doubled fluxes with halved steps take none (step of 256^3 FP32
// 2.059 ms, 2.066 so; 384^3 with HSE 8.89, 8.95), but the limiter's products then
// leave FP32 at flux differences of 0.9e19 already, not 1.3e19.
template <typename T, bool HSE>
struct CellQ {
  T u[5];
  T F[5];
  T vd, cF, d;
  T cS, xiE;
  T sup;  // 1 where |v| > c_S (the limiter switch of Sect. 2.2), else 0
};

// Half the flux; the mass flux is the momentum, which is not kept twice.
template <int D, typename T, bool HSE>
__device__ __forceinline__ T half_flux(const CellQ<T, HSE>& c, int i) {
  return i == RHO ? T(0.5) * c.u[MX + D] : c.F[i];
}

// E = rho e + m^2/(2 rho) + b^2/2 and p = (gamma-1) rho e (Sect. 2.1, Eq. 5):
// the cancellation step, always evaluated in FP64.
template <typename T>
__device__ __forceinline__ T pressure(const T* u, double b2, double gm1) {
  const double rho = (double)u[RHO];
  const double mx = (double)u[MX], my = (double)u[MY], mz = (double)u[MZ];
  const double m2 = mx * mx + my * my + mz * mz;
  const double ri = rinv64(rho, u[RHO]);
  return (T)(gm1 * ((double)u[EN] - 0.5 * m2 * ri - 0.5 * b2));
}

// Directional fast magnetosonic speed (named after Eq. 21) from q = a^2 +
// b^2/rho: c_F^2 = q/2 + sqrt((q/2)^2 - a^2 b_d^2/rho).
template <typename T>
__device__ __forceinline__ T fast_speed(T q, T a2, T bd, T ri) {
  const T h = T(0.5) * q;
  return fsqrt(h + fsqrt(nonneg(h * h - a2 * bd * bd * ri)));
}

template <typename T, int D, bool HSE>
__device__ __forceinline__ void cell_quantities(const T* u, const FieldQ<T>& f, double gamma, CellQ<T, HSE>& c) {
#pragma unroll
  for (int k = 0; k < 5; ++k) c.u[k] = u[k];
  const T ri = rcp(u[RHO]), hri = T(0.5) * ri;
  const T hv[3] = {u[MX] * hri, u[MY] * hri, u[MZ] * hri};
  const T p = pressure<T>(u, f.b2, gamma - 1.0);
  const T b2 = (T)f.b2;
  const T ptot = p + T(0.5) * b2;
  const T a2 = (T)gamma * p * ri;
  const T q = a2 + b2 * ri;
  const T hbv = f.b[0] * hv[0] + f.b[1] * hv[1] + f.b[2] * hv[2];
  const T cf = fast_speed(q, a2, f.b[D], ri);
  const T md = u[MX + D], hb = T(0.5) * f.b[D];
  c.F[RHO] = T(0);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    T x = md * hv[k] - hb * f.b[k];
    if (k == D) x += T(0.5) * ptot;
    c.F[MX + k] = x;
  }
  c.F[EN] = (u[EN] + ptot) * hv[D] - f.b[D] * hbv;
  c.vd = hv[D];
  c.cF = HSE ? T(0.5) * cf : T(0);
  c.d = fabs(hv[D]) + T(0.5) * cf;
  c.sup = T(4) * (hv[0] * hv[0] + hv[1] * hv[1] + hv[2] * hv[2]) > a2 ? T(1) : T(0);
  if (HSE) {
    c.cS = fsqrt(a2);
    c.xiE = -(u[EN] + p);
  } else {
    c.cS = T(0);
    c.xiE = T(0);
  }
}

// Limiters, Eqs. (29)-(30).  minmod as the median of a, b and 0 (of finite
// operands; with a NaN the FP32 instruction gives the least of the other two).
// No product that could underflow decides the sign.
__device__ __forceinline__ float minmod(float a, float b) { return __builtin_amdgcn_fmed3f(a, b, 0.0f); }
__device__ __forceinline__ double minmod(double a, double b) {
  return fmax(fmin(a, b), 0.0) + fmin(fmax(a, b), 0.0);
}
// Half the van Leer limiter, the harmonic mean ab/(a+b) where a and b share a
// sign (the printed sign prefactor would flip negative pairs), else 0.
template <typename T>
__device__ __forceinline__ T half_vanleer(T a, T b) {
  // the quotient is formed unconditionally and selected: as an arm of the
  // conditional, the FP64 reciprocal's length would keep it a branch
  const T ab = a * b;
  const T q = ab * rcp(a + b);
  return ab > T(0) ? q : T(0);
}
// The limited value of a and b, LIM 0 minmod, 1 van Leer, 2 the switch of
// Sect. 2.2 (minmod where the cell is supersonic, sup = 1; van Leer elsewhere),
// as the cheapest multiple of it: limit_unit<LIM>() times the result is the
// limited value.
template <typename T, int LIM>
__device__ __forceinline__ T limit_scaled(T sup, T a, T b) {
  if (LIM == 0) return minmod(a, b);
  if (LIM == 1) return half_vanleer(a, b);
  return sup != T(0) ? T(0.5) * minmod(a, b) : half_vanleer(a, b);
}
template <int LIM>
__device__ constexpr int limit_unit() {
  return LIM == 0 ? 1 : 2;
}

// The gradient scale of the hydrostatic correction as a finite number.  A
// negative pressure of a half-step state has no sound speed; its NaN would reach
// minmod, where the FP32 median gives the lesser of du and 0, not du (as the FP64
// form does).  With 0 in its place du is the limited value.  An infinite scale
// (a pressure of zero) becomes the largest number: minmod decides alike, and
// times a zero xi it is 0.
__device__ __forceinline__ float finite_scale(float s) {
  return s == s ? __builtin_amdgcn_fmed3f(s, -3.402823466e38f, 3.402823466e38f) : 0.0f;
}
__device__ __forceinline__ double finite_scale(double s) { return s; }

// Dissipation Q_j at the interface between cells L and R, so that the
// first-order relaxed flux is F_L + F_R - Q_j with the half fluxes and speeds:
//   no HSE: Q = max(d_L, d_R) (u_R - u_L), Eqs. (24)-(25);
//   HSE:    Q = max(|v_L|, |v_R|) du + max(cF_L, cF_R) minmod(du - g, du),
//           g = (xi_L + xi_R)/2 (phi_R - phi_L)/(cS_L cS_R), Eqs. (50)-(57).
template <typename T, bool HSE>
__device__ __forceinline__ void dissipation(const CellQ<T, HSE>& L, const CellQ<T, HSE>& R, T phiL, T phiR,
                                            T* Q) {
  if (!HSE) {
    const T dmax = speed_max(L.d, R.d);
#pragma unroll
    for (int k = 0; k < 5; ++k) Q[k] = dmax * (R.u[k] - L.u[k]);
  } else {
    const T avL = fabs(L.vd), avR = fabs(R.vd);
    const T dadv = speed_max(avL, avR);
    const T dac = speed_max(L.cF, R.cF);
    const T scale = finite_scale(T(0.5) * ((phiR - phiL) * rcp(L.cS * R.cS)));  // (exact: the mean of xi taken here)
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      const T du = R.u[k] - L.u[k];
      const T xiL = (k == EN) ? L.xiE : -L.u[k];
      const T xiR = (k == EN) ? R.xiE : -R.u[k];
      const T g = (xiL + xiR) * scale;
      const T delta = minmod(du - g, du);
      Q[k] = dadv * du + dac * delta;
    }
  }
}

// Unsplit gravitational source of cell i, Eq. (42) with the sign of Eq. (36):
// S = -(0, rho e_D, m_D) (phi_i+1 - phi_i-1)/(2 h); inv2h = 1/(2 h).
template <typename T, int D>
__device__ __forceinline__ void gravity_source(T rho, T mD, T dphi2, T inv2h, T* S) {
  const T gr = dphi2 * inv2h;
#pragma unroll
  for (int k = 0; k < 5; ++k) S[k] = T(0);
  S[MX + D] = -rho * gr;
  S[EN] = -mD * gr;
}

// Split gravity G_D over half a step, Eqs. (39)-(40): m_D -= rho gh with
// gh = (dt/2)(phi_i+1 - phi_i-1)/(2 h).  Density and internal energy stay, so
// E changes by the kinetic energy, (m'^2 - m^2)/(2 rho) = -gh (m + m')/2.
template <typename T, int D>
__device__ __forceinline__ void gravity_kick(T* u, T gh) {
  const T m = u[MX + D];
  const T mn = m - u[RHO] * gh;
  u[MX + D] = mn;
  u[EN] = u[EN] - gh * (T(0.5) * (m + mn));
}

// ----------------------------------------------------------- index maps
// Periodic axes wrap; outflow axes copy the nearest real entry (zeroth-order
// extrapolation).  A face array along its own normal has n+1 real faces on
// an outflow axis (last real face n) and n on a periodic one.
__device__ __forceinline__ int wrap(int i, int n) {
  if (i >= 0 && i < n) return i;
  int r = i % n;
  return r < 0 ? r + n : r;
}
__device__ __forceinline__ int map_cell(int i, int n, int bc) {
  if (i >= 0 && i < n) return i;
  if (bc == 0) return wrap(i, n);
  return i < 0 ? 0 : n - 1;
}
__device__ __forceinline__ int map_face(int i, int n, int bc) {
  if (bc == 0) return wrap(i, n);
  return i < 0 ? 0 : (i > n ? n : i);
}

}  // namespace fish
