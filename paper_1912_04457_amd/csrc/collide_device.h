// Monte Carlo collision term (Eq. C_a_b, Eq. MC C_gg, Eq. small c relation).
//
// Work item = (cell, channel, observed node p1).  A wavefront works on one item
// at a time (where items are few, several wavefronts on parts of its samples),
// so everything that depends only on the item (p1, E1, f1, masses, channel) is
// wave-uniform; the 64 lanes draw samples s = lane, lane+64, ...
//
// Per sample (CM-angle parameterisation of the 5-D integral):
//   Philox4x32-10 block -> five 23-bit uniforms -> p2 in the box, cos theta*,
//   phi* -> E2, s, |p*| -> k1 boosted to the CM frame gives the polar axis ->
//   p3* on the sphere -> boost back, p4 = P - p3 -> box cut -> t, u ->
//   |M|^2 (Table I) -> trilinear f at p2, p3, p4 -> bracket
//   B = f3 f4 F1 F2 - f1 f2 F3 F4 -> value v.
// Symmetric sampling adds +v at (X, p1), +v W(p2) at species 2, -v W(p3) at
// species 3 and -v W(p4) at species 4 (W: trilinear stencil weights).
//
// Precision: the sample geometry (everything that decides the threshold,
// the box cut and the branch of the CM frame) is FP64 in both modes, so both
// precisions reject exactly the samples an FP64 evaluation rejects; on CDNA4
// FP64 add/mul/FMA issue at the rate of unpacked FP32.  The integrand
// (|M|^2, interpolation, bracket, value) is FP32 in QGBE_FP32 mode.  Direct
// sums and deposits are FP64 in both modes.
#pragma once

#include <hip/hip_runtime.h>

#include "collide.h"

namespace qgbe {
namespace {

constexpr int kWave = 64;

__device__ __forceinline__ double unif23(uint32_t v) { return ((double)v + 0.5) * (1.0 / 8388608.0); }

// FP64 1/x and 1/sqrt(x) for finite x > 0: the hardware estimate (measured
// relative error below 2^-24 on gfx950) refined by one third-order step,
// which leaves ~2^-72 (below the last bit) without the scaling and
// special-case handling of a general division or square root.
//   1/x:       e = 1 - x r,          r (1 + e + e^2)
//   1/sqrt(x): t = (1 - x y^2) / 2,  y (1 + t + 3/2 t^2)
__device__ __forceinline__ double rcp64(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, r, 1.0);
  return fma(r, fma(e, e, e), r);
}

__device__ __forceinline__ double rsqrt64(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double t = fma(-0.5 * x * y, y, 0.5);
  return fma(y, fma(1.5 * t, t, t), y);
}

__device__ __forceinline__ double sqrt64(double x) { return x > 0.0 ? x * rsqrt64(x) : 0.0; }

// sqrt(x) for finite x > 0, refined as rsqrt64: g = x y, r = (1 - g y) / 2,
// g (1 + r + 3/2 r^2).
__device__ __forceinline__ double sqrt_pos(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double g = x * y;
  const double r = fma(-0.5 * g, y, 0.5);
  return fma(g, fma(1.5 * r, r, r), g);
}

// x with its sign flipped where bit 31 of m is set.
__device__ __forceinline__ double flip_sign(double x, uint32_t m) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(x);
  return __longlong_as_double((long long)(b ^ ((unsigned long long)(m & 0x80000000u) << 32)));
}

// a b + c with a constant c.  Written out, the compiler keeps the coefficients
// of the polynomials below in vector registers (26 to 64 of the 168) and copies
// each before the accumulating form of the instruction overwrites it; in a
// scalar pair c costs neither (scalar moves issue beside the vector unit).
__device__ __forceinline__ double fma_k(double a, double b, double c) {
  double d;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(c));
  return d;
}

// sin(pi r) and cos(pi r) for |r| <= 1/4, moved to the quadrant k (mod 4):
// sin(pi r) = r S(r^2) and cos(pi r) = C(r^2) with S and C of degree 6
// (Chebyshev-node fits, gen_fp64_poly.py; fit errors 1e-17 and 5e-17).
// Measured on the CPU over every 23-bit u: within 1.8e-16 of sin and cos (the
// Taylor series to r^15 and r^16 they replace: 1.9e-16).
__device__ __forceinline__ void sincos_quadrant(double r, int k, double& sn, double& cs) {
  const double r2 = r * r;
  double ps = 0.0004615313805851339;
  ps = fma_k(ps, r2, -0.0073700215052934955);
  ps = fma_k(ps, r2, 0.08214586917478434);
  ps = fma_k(ps, r2, -0.5992645289394928);
  ps = fma_k(ps, r2, 2.550164039873374);
  ps = fma_k(ps, r2, -5.167712780049954);
  ps = fma_k(ps, r2, 3.141592653589793);
  ps *= r;
  double pc = 0.001906807054314109;
  pc = fma_k(pc, r2, -0.025804938121446575);
  pc = fma_k(pc, r2, 0.23533054718578558);
  pc = fma_k(pc, r2, -1.3352627670358546);
  pc = fma_k(pc, r2, 4.058712126397826);
  pc = fma_k(pc, r2, -4.934802200544605);
  pc = fma(pc, r2, 1.0);
  const double a = (k & 1) ? pc : ps;   // sin before the sign
  const double b = (k & 1) ? ps : pc;   // cos before the sign
  sn = flip_sign(a, (uint32_t)k << 30);
  cs = flip_sign(b, (uint32_t)(k + 1) << 30);
}

// sin and cos of 2 pi u for u in [0, 1): 2u = k/2 + r, k the nearest integer
// to 4u (exact: u has at most 24 significant bits, or r's rounding is below
// the fits' errors).
__device__ __forceinline__ void sincos_2pi(double u, double& sn, double& cs) {
  const double q = rint(4.0 * u);
  sincos_quadrant(fma(-0.5, q, 2.0 * u), (int)q, sn, cs);
}

// The same for u = (v + 1/2) 2^-23: the quadrant and the remainder are bit
// fields of v.
__device__ __forceinline__ void sincos_2pi_23(uint32_t v, double& sn, double& cs) {
  const int rem = (int)(v << 11) >> 11;  // the low 21 bits, signed
  sincos_quadrant(fma((double)rem, 0x1p-22, 0x1p-23), (int)((v + (1u << 20)) >> 21), sn, cs);
}

// e^x: x = k ln2 + r with |r| <= ln2/2 (ln2 split so k*ln2_hi is exact for
// |k| < 2^11), e^r = 1 + r (1 + r g(r)) with g of degree 9 (a Chebyshev-node
// fit, gen_fp64_poly.py; relative error of e^r from the fit 2e-17), times
// 2^k.  Overflows to inf and underflows to 0 like exp.  Measured on the CPU:
// within 0.95 ulp over |x| < 700 (the Taylor series to r^13 it replaces: 0.89).
__device__ __forceinline__ double exp64(double x) {
  const double k = rint(x * 1.4426950408889634);
  double r = fma(-k, 0.6931471805598903, x);
  r = fma(-k, 5.497923018708371e-14, r);
  double p = 2.510038549551032e-08;
  p = fma_k(p, r, 2.7620088445409746e-07);
  p = fma_k(p, r, 2.7557268459997064e-06);
  p = fma_k(p, r, 2.4801521295954376e-05);
  p = fma_k(p, r, 0.00019841269863053618);
  p = fma_k(p, r, 0.0013888888917213717);
  p = fma_k(p, r, 0.008333333333330062);
  p = fma_k(p, r, 0.04166666666662413);
  p = fma_k(p, r, 0.16666666666666669);
  p = fma_k(p, r, 0.5000000000000001);
  p = fma(p, r, 1.0);
  p = fma(p, r, 1.0);
  return ldexp(p, (int)k);
}

// ln a for finite a > 0: a = m 2^e with m in [1/sqrt2, sqrt2), ln m =
// 2 atanh(s) = 2 s P(s^2), s = (m-1)/(m+1), |s| <= 0.172, P of degree 7 (a
// Chebyshev-node fit of atanh(sqrt w)/sqrt w, gen_fp64_poly.py; relative
// fit error 1e-18).  Measured on the CPU: within 2.1 ulp of ln on the 23-bit
// uniforms, 2.7 ulp elsewhere (the series to s^21 it replaces: the same).
__device__ __forceinline__ double log64(double a) {
  int e;
  double m = frexp(a, &e);
  if (m < 0.7071067811865476) {
    m *= 2.0;
    e -= 1;
  }
  const double s = (m - 1.0) * rcp64(m + 1.0);
  const double s2 = s * s;
  double p = 0.07404933786156531;
  p = fma_k(p, s2, 0.0765625655736915);
  p = fma_k(p, s2, 0.09091816120808513);
  p = fma_k(p, s2, 0.11111098523202137);
  p = fma_k(p, s2, 0.1428571438036914);
  p = fma_k(p, s2, 0.19999999999650955);
  p = fma_k(p, s2, 0.33333333333333826);
  p = fma(p, s2, 1.0);
  const double de = (double)e;
  return fma(de, 0.6931471805598903, fma(de, 5.497923018708371e-14, 2.0 * s * p));
}


template <typename R>
__device__ __forceinline__ R rcp_r(R x);
template <>
__device__ __forceinline__ float rcp_r<float>(float x) { return __builtin_amdgcn_rcpf(x); }
template <>
__device__ __forceinline__ double rcp_r<double>(double x) { return rcp64(x); }

// Table I |M|^2 in units of g^4, every t and u pole regulated by mu = m_g^2.
// Group factors (SU(3), fundamental quarks): 8 dF^2 CF^2/dA = 16,
// 16 dF CF (CF - CA/2) = -32/3, 8 dF CF^2 = 128/3, 8 dF CF CA = 96,
// 16 dA CA^2 = 1152.
template <typename R>
__device__ __forceinline__ R matrix_element(int row, R s, R t, R u, R mu) {
  const R rt = rcp_r<R>(t - mu);
  const R ru = rcp_r<R>(u - mu);
  const R rs = rcp_r<R>(s);
  const R s2 = s * s, t2 = t * t, u2 = u * u;
  switch (row) {
    case 1: return R(16) * (s2 + u2) * rt * rt;
    case 2: return R(16) * ((s2 + u2) * rt * rt + (s2 + t2) * ru * ru) - R(32.0 / 3.0) * s2 * rt * ru;
    case 3: return R(16) * ((s2 + u2) * rt * rt + (u2 + t2) * rs * rs) - R(32.0 / 3.0) * u2 * rt * rs;
    case 4: return R(16) * (t2 + u2) * rs * rs;
    case 5: return R(128.0 / 3.0) * (u * rt + t * ru) - R(96) * (t2 + u2) * rs * rs;
    case 6: return R(-128.0 / 3.0) * (u * rs + s * ru) + R(96) * (s2 + u2) * rt * rt;
    default: return R(1152) * (R(3) - s * u * rt * rt - s * t * ru * ru - t * u * rs * rs);
  }
}

// |M|^2 / g^4 of a row: the user's terms where the row was replaced (the
// row is uniform over a wavefront), else Table I.
// kUser = false: no user terms in this launch (the table's rows only).
template <typename R, bool kUser = true>
__device__ __forceinline__ R msq_row(uint32_t mask, const MsqTable* tab, int row, R s, R t, R u, R mu) {
  if (!kUser || !((mask >> row) & 1u)) return matrix_element<R>(row, s, t, u, mu);
  const R x[6] = {s, t, u, rcp_r<R>(t - mu), rcp_r<R>(u - mu), rcp_r<R>(s)};
  R sum = R(0);
  const int n = tab->n[row];
  for (int k = 0; k < n; ++k) {
    R term = (R)tab->c[row][k];
    for (int i = 0; i < 6; ++i)
      for (int e = 0; e < tab->p[row][k][i]; ++e) term *= x[i];
    sum += term;
  }
  return sum;
}

// Trilinear stencil over the 8 surrounding cell centres, clamped at the box.
template <typename R>
struct Stencil {
  int base;
  R wx, wy, wz;
};

// The grid coordinate and its fraction are formed in FP64 so the weights carry
// a relative (not an absolute 2^-24 * n) error when rounded to R.
// (FP32 weights: the largest coordinate below n - 1 stands for n - 1, so the
// whole part is at most n - 2 by itself, and the fraction rounds to 1.)
template <typename R>
__device__ __forceinline__ R clamp_axis(double p, double pc, double inv_dp, int n, int& i0) {
  if constexpr (sizeof(R) == sizeof(float)) {
    const double top = __longlong_as_double(__double_as_longlong((double)(n - 1)) - 1);
    const double t = fmin(fmax(fma(p, inv_dp, pc), 0.0), top);
    i0 = (int)t;
    return (R)__builtin_amdgcn_fract(t);
  }
  const double t = fmin(fmax(fma(p, inv_dp, pc), 0.0), (double)(n - 1));
  const int i = min((int)t, n - 2);
  i0 = i;
  return (R)(t - (double)i);
}

template <typename R>
__device__ __forceinline__ Stencil<R> make_stencil(const double p[3], const Grid& G) {
  Stencil<R> st;
  int ix, iy, iz;
  st.wx = clamp_axis<R>(p[0], G.pc[0], G.inv_dp[0], G.np[0], ix);
  st.wy = clamp_axis<R>(p[1], G.pc[1], G.inv_dp[1], G.np[1], iy);
  st.wz = clamp_axis<R>(p[2], G.pc[2], G.inv_dp[2], G.np[2], iz);
  st.base = ix * G.ox + iy * G.oy + iz;
  return st;
}

template <typename R, typename T>
__device__ __forceinline__ R interpolate(const T* __restrict__ tile, const Stencil<R>& st, int ox, int oy) {
  const T* q = tile + st.base;
  const R f000 = q[0], f001 = q[1], f010 = q[oy], f011 = q[oy + 1];
  const R f100 = q[ox], f101 = q[ox + 1], f110 = q[ox + oy], f111 = q[ox + oy + 1];
  const R a00 = f000 + st.wz * (f001 - f000);
  const R a01 = f010 + st.wz * (f011 - f010);
  const R a10 = f100 + st.wz * (f101 - f100);
  const R a11 = f110 + st.wz * (f111 - f110);
  const R b0 = a00 + st.wy * (a01 - a00);
  const R b1 = a10 + st.wy * (a11 - a10);
  return b0 + st.wx * (b1 - b0);
}

// Scatter v with the stencil weights (the transpose of interpolate): values
// in precision R, accumulators of type T.  kScope selects the atomic's memory
// scope: workgroup for accumulators in LDS, agent for global memory (the two
// kinds stay distinct instructions, so each keeps its address space).
template <typename R, typename T, int kScope = __HIP_MEMORY_SCOPE_AGENT>
__device__ __forceinline__ void deposit(T* acc, const Stencil<R>& st, R v, int ox, int oy) {
  T* q = acc + st.base;
  const R vx1 = v * st.wx, vx0 = v - vx1;
  const R v01 = vx0 * st.wy, v00 = vx0 - v01;
  const R v11 = vx1 * st.wy, v10 = vx1 - v11;
  __hip_atomic_fetch_add(q, (T)(v00 - v00 * st.wz), __ATOMIC_RELAXED, kScope);
  __hip_atomic_fetch_add(q + 1, (T)(v00 * st.wz), __ATOMIC_RELAXED, kScope);
  __hip_atomic_fetch_add(q + oy, (T)(v01 - v01 * st.wz), __ATOMIC_RELAXED, kScope);
  __hip_atomic_fetch_add(q + oy + 1, (T)(v01 * st.wz), __ATOMIC_RELAXED, kScope);
  __hip_atomic_fetch_add(q + ox, (T)(v10 - v10 * st.wz), __ATOMIC_RELAXED, kScope);
  __hip_atomic_fetch_add(q + ox + 1, (T)(v10 * st.wz), __ATOMIC_RELAXED, kScope);
  __hip_atomic_fetch_add(q + ox + oy, (T)(v11 - v11 * st.wz), __ATOMIC_RELAXED, kScope);
  __hip_atomic_fetch_add(q + ox + oy + 1, (T)(v11 * st.wz), __ATOMIC_RELAXED, kScope);
}

// The same deposit into accumulators that cover only the nodes [lo, lo + n)
// (acc[0] is node lo): the same corner values; a corner outside the window
// is left to the launch whose window holds it.
__device__ __forceinline__ void deposit_window(double* acc, const Stencil<double>& st, double v, int ox, int oy,
                                               int lo, int n) {
  const int b = st.base - lo;
  const double vx1 = v * st.wx, vx0 = v - vx1;
  const double v01 = vx0 * st.wy, v00 = vx0 - v01;
  const double v11 = vx1 * st.wy, v10 = vx1 - v11;
  const int off[8] = {0, 1, oy, oy + 1, ox, ox + 1, ox + oy, ox + oy + 1};
  const double val[8] = {v00 - v00 * st.wz, v00 * st.wz, v01 - v01 * st.wz, v01 * st.wz,
                         v10 - v10 * st.wz, v10 * st.wz, v11 - v11 * st.wz, v11 * st.wz};
#pragma unroll
  for (int c = 0; c < 8; ++c)
    if ((unsigned)(b + off[c]) < (unsigned)n)
      __hip_atomic_fetch_add(acc + b + off[c], val[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// 1 / ((2 pi)^3 * 2 * 2 * 16 pi^2): two-body phase space |p*|/(16 pi^2 sqrt s),
// k2 measure d^3k2/((2 pi)^3 2 E2) and 1/(2 E1) of Eq. C_a_b
constexpr double kNorm = 1.0 / (8.0 * kPi * kPi * kPi * 4.0 * 16.0 * kPi * kPi);

// Quantities of a work item, identical for all lanes of the wave.
struct Item {
  int cell, p1_lin;
  double p1[3];
  double E1;
  double m1sq, m2sq, m3sq, m4sq;
  double dm34;              // m3^2 - m4^2
  double dde, sde;          // m1^2 - m2^2 -+ dm34: E1* -+ ... of t and u, times 2 sqrt s
  double sum2, dif2;        // (m3 + m4)^2 (the threshold of s), (m3 - m4)^2
  double mu;                // regulator m_g^2
  double f1;
  double coef;              // w V5 / N (symmetric) or sigma V5 / N (direct)
  double pref;              // coef g^4 / ((2pi)^3 4 16 pi^2 E1): item part of the value
};

// The sampled configuration (FP64 geometry).
struct Geo {
  double p2[3], p3[3], p4[3];
  double E2, s, t, u, rs, pstar;
};

// Where a sample lies: p2 in the box, cos and sin of theta* (and 2 (1 -+ cos)
// for t and u, without cancellation), cos and sin of phi*.
struct SampleMap {
  double p2[3], cth, sth, omc2, opc2, cphi, sphi;
};

// From the five unit-cube variables (the mixture's; any doubles in (0, 1)).
__device__ __forceinline__ SampleMap map_unit(const Grid& G, const double u[5]) {
  SampleMap m;
  for (int a = 0; a < 3; ++a) m.p2[a] = fma(2.0 * G.ph[a], u[a], -G.ph[a]);
  const double w = 1.0 - u[3];
  m.cth = fma(2.0, u[3], -1.0);
  m.sth = 2.0 * sqrt64(u[3] * w);
  m.omc2 = 4.0 * w;
  m.opc2 = 4.0 * u[3];
  sincos_2pi(u[4], m.sphi, m.cphi);
  return m;
}

// Five 23-bit uniforms (v + 1/2) 2^-23 from one Philox block: the top 23 bits
// of each word, and for the fifth the low 9 bits of words 0 and 1 and bits
// 4..8 of word 2.
__device__ __forceinline__ uint32_t fifth_word(uint32_t x0, uint32_t x1, uint32_t x2) {
  return ((x0 & 0x1FFu) << 14) | ((x1 & 0x1FFu) << 5) | ((x2 & 0x1FFu) >> 4);
}

__device__ __forceinline__ void five_uniforms(uint32_t x0, uint32_t x1, uint32_t x2, uint32_t x3, double u[5]) {
  u[0] = unif23(x0 >> 9);
  u[1] = unif23(x1 >> 9);
  u[2] = unif23(x2 >> 9);
  u[3] = unif23(x3 >> 9);
  u[4] = unif23(fifth_word(x0, x1, x2));
}

// 2 (v + 1/2) 2^-23 - 1, exact.
__device__ __forceinline__ double centred23(uint32_t v) { return fma((double)v, 0x1p-22, 0x1p-23 - 1.0); }

// The uniform sampler's map, straight from the words.
__device__ __forceinline__ SampleMap map_words(const Grid& G, uint32_t x0, uint32_t x1, uint32_t x2, uint32_t x3) {
  SampleMap m;
  m.p2[0] = G.ph[0] * centred23(x0 >> 9);
  m.p2[1] = G.ph[1] * centred23(x1 >> 9);
  m.p2[2] = G.ph[2] * centred23(x2 >> 9);
  m.cth = centred23(x3 >> 9);
  m.sth = sqrt_pos(fma(-m.cth, m.cth, 1.0));
  m.omc2 = fma(-2.0, m.cth, 2.0);
  m.opc2 = fma(2.0, m.cth, 2.0);
  sincos_2pi_23(fifth_word(x0, x1, x2), m.sphi, m.cphi);
  return m;
}

// Sample geometry; false if below threshold or outside the box.  FP64 and the
// bound of every sampler's loop (VALU issue), so written for few operations:
// p3* = p* (sin cos phi e1 + sin sin phi e2 + cos n) with the frame of n
// multiplied out, and t and u from the CM frame, t = (E1* - E3*)^2 - (p1* -
// p*)^2 - 2 p1* p* (1 - cos), u likewise with E4* and 1 + cos: E1* - E3* and
// E1* - E4* are mass differences over 2 sqrt s, and a small t or u keeps its
// relative accuracy (differences of momenta lose it).  With the constants of
// the polynomials in scalar registers, the three-way xors and map_words, a term
// of 256 cells x 8000 nodes x 2048 samples takes 59.8 ms where the plain form
// (frame vectors, t and u from the lab momenta) took 66.8; 7 species x 17
// channels x 8000 x 4096 mixture samples 7.36 for 7.84.
__device__ __forceinline__ bool geometry(const Item& it, const Grid& G, const SampleMap& m, Geo& g) {
  for (int a = 0; a < 3; ++a) g.p2[a] = m.p2[a];
  g.E2 = sqrt_pos(g.p2[0] * g.p2[0] + g.p2[1] * g.p2[1] + g.p2[2] * g.p2[2] + it.m2sq);  // p2 = 0, m2 = 0: NaN, rejected below
  const double E = it.E1 + g.E2;
  const double P[3] = {it.p1[0] + g.p2[0], it.p1[1] + g.p2[1], it.p1[2] + g.p2[2]};
  const double s = E * E - (P[0] * P[0] + P[1] * P[1] + P[2] * P[2]);
  g.s = s;
  if (!(s > it.sum2)) return false;  // threshold (m3 + m4)^2
  const double rs = rsqrt64(s);
  const double sq = s * rs, hrs = 0.5 * rs;
  g.rs = rs;
  g.pstar = hrs * sqrt_pos((s - it.sum2) * (s - it.dif2));
  // k1 in the CM frame: p1* = p1 + P ((P.p1)/(sqrt s (E + sqrt s)) - E1/sqrt s)
  const double inv_E = rcp64(E + sq);
  const double Pp1 = P[0] * it.p1[0] + P[1] * it.p1[1] + P[2] * it.p1[2];
  const double c1 = (Pp1 * inv_E - it.E1) * rs;
  double n[3] = {it.p1[0] + P[0] * c1, it.p1[1] + P[1] * c1, it.p1[2] + P[2] * c1};
  const double nn = n[0] * n[0] + n[1] * n[1] + n[2] * n[2];
  const double rn = rsqrt64(nn);
  n[0] *= rn; n[1] *= rn; n[2] *= rn;
  // orthonormal completion of n (Duff et al., JCGT 6(1), 2017): with sg the
  // sign of n_z, a = -1 / (sg + n_z), e1 = (1 + sg n_x^2 a, sg n_x n_y a, -sg n_x)
  // and e2 = (n_x n_y a, sg + n_y^2 a, -n_y)
  const uint32_t sgn = (uint32_t)((unsigned long long)__double_as_longlong(n[2]) >> 32);
  const double ra = rcp64(flip_sign(1.0, sgn) + n[2]);
  const double st = m.sth * g.pstar, ct = m.cth * g.pstar;
  const double sc = st * m.cphi, ss = st * m.sphi;
  const double w = fma(flip_sign(sc, sgn), n[0], ss * n[1]);
  const double c2 = fma(-ra, w, ct);
  const double p3s[3] = {fma(n[0], c2, sc), fma(n[1], c2, flip_sign(ss, sgn)), fma(n[2], ct, -w)};
  const double E3s = (s + it.dm34) * hrs;
  const double Pp3 = P[0] * p3s[0] + P[1] * p3s[1] + P[2] * p3s[2];
  const double c3 = (Pp3 * inv_E + E3s) * rs;
  for (int k = 0; k < 3; ++k) {
    g.p3[k] = p3s[k] + P[k] * c3;
    g.p4[k] = P[k] - g.p3[k];
  }
  for (int k = 0; k < 3; ++k) {
    if (!(fabs(g.p3[k]) <= G.ph[k]) || !(fabs(g.p4[k]) <= G.ph[k])) return false;
  }
  const double p1s = nn * rn, pp = p1s * g.pstar;
  const double dp = p1s - g.pstar, dp2 = dp * dp;
  const double d3 = it.dde * hrs, d4 = it.sde * hrs;
  g.t = fma(-pp, m.omc2, fma(d3, d3, -dp2));
  g.u = fma(-pp, m.opc2, fma(d4, d4, -dp2));
  return true;
}

// Order a wave's LDS accesses across its lanes (the LDS executes one wave's
// instructions in order; this keeps the compiler from reordering them).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Wavefront sums.  The short-item form uses DPP: two quad permutations and two rotations within
// each 16-lane row leave every lane with its row's sum; the four row sums
// are read from lanes 0, 16, 32, 48 and added in a fixed order.  Every lane
// must be active.
template <int kCtrl>
__device__ __forceinline__ int dpp_i32(int v) {
  return __builtin_amdgcn_update_dpp(0, v, kCtrl, 0xF, 0xF, false);
}

template <int kCtrl>
__device__ __forceinline__ double dpp_f64(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = (unsigned)dpp_i32<kCtrl>((int)(unsigned)b);
  const unsigned hi = (unsigned)dpp_i32<kCtrl>((int)(unsigned)(b >> 32));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

__device__ __forceinline__ double readlane_f64(double v, int lane) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, lane);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), lane);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Butterfly sums through lane permutes, for the long-item form.
__device__ __forceinline__ int wave_count(int v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
  return v;
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
  return v;
}

__device__ __forceinline__ int wave_count_dpp(int v) {
  v += dpp_i32<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp_i32<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp_i32<0x124>(v);  // row_ror:4
  v += dpp_i32<0x128>(v);  // row_ror:8
  return (__builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16)) +
         (__builtin_amdgcn_readlane(v, 32) + __builtin_amdgcn_readlane(v, 48));
}

__device__ __forceinline__ double wave_sum_dpp(double v) {
  v += dpp_f64<0xB1>(v);
  v += dpp_f64<0x4E>(v);
  v += dpp_f64<0x124>(v);
  v += dpp_f64<0x128>(v);
  return (readlane_f64(v, 0) + readlane_f64(v, 16)) + (readlane_f64(v, 32) + readlane_f64(v, 48));
}

// ---------------------------------------------------------------------------
// Mixture proposal (learned sampler).  Row = (channel, observed node).
// thr[0] = alpha 2^32 selects the defensive uniform component; component k is
// drawn when thr[k] <= x < thr[k+1].  Its five coordinates are logistic-normal:
// y = mu + sigma z (z from Box-Muller), u = 1/(1 + exp(-y)).  The sample
// location is formed in FP64 (it decides the threshold and the box cut); the
// density q(u) = alpha + sum_k pi_k prod_d N(y_d; mu, sigma)/(u_d(1-u_d)) is
// evaluated in the kernel's precision.
// ---------------------------------------------------------------------------
constexpr double kTwo32 = 4294967296.0;
constexpr double kHalfLog2Pi = 0.91893853320467274178;

// Per-item constants of the FP32 sampler, one row per wave in LDS: mu (40),
// 1/sigma (40), log pi_k - sum_d log sigma_kd - 5/2 log 2 pi (8), alpha,
// sigma (40).
constexpr int kMixSigma = 89;
constexpr int kMixRow = kMixSigma + 40;
static_assert(5 * kMixKF32 == 40 && kMixKF32 <= 8, "row layout: 8 components");

// The same draw for the FP32 kernel: component parameters from the wave's
// LDS row (see mix_prepare_f32), thresholds from the (wave-uniform) table
// row; u in FP64 (it feeds the FP64 geometry), y in FP32 (it feeds only the
// FP32 density).
__device__ __forceinline__ void mix_draw_row(const uint32_t x[8], const uint32_t* __restrict__ thr, const float* row,
                                             int K, double u[5], float y[5]) {
  if (x[0] < thr[0]) {
    for (int d = 0; d < 5; ++d) {
      const uint32_t v = x[1 + d] >> 9;
      u[d] = unif23(v);
      const float uf = ((float)v + 0.5f) * (1.0f / 8388608.0f);  // = u[d] exactly, >= 2^-24
      // logit u = ln 2 (log2 u - log2 (1 - u)); v_log_f32 is log2 (no denormals here)
      y[d] = 0.6931471805599453f * (__builtin_amdgcn_logf(uf) - __builtin_amdgcn_logf(1.0f - uf));
    }
    return;
  }
  // component: the last threshold at or below x[0] (unrolled to the 8
  // components this row layout holds, so the threshold loads issue together)
  int k = 0;
#pragma unroll
  for (int j = 1; j < kMixKF32; ++j)
    if (j < K) k = x[0] >= thr[j] ? j : k;
  double z[6];
  for (int pr = 0; pr < 3; ++pr) {
    const double a1 = unif23(x[1 + 2 * pr] >> 9), a2 = unif23(x[2 + 2 * pr] >> 9);
    const double r = sqrt64(-2.0 * log64(a1));
    double sn, cs;
    sincos_2pi(a2, sn, cs);
    z[2 * pr] = r * cs;
    z[2 * pr + 1] = r * sn;
  }
  for (int d = 0; d < 5; ++d) {
    const double yd = (double)row[k * 5 + d] + (double)row[kMixSigma + k * 5 + d] * z[d];
    u[d] = rcp64(1.0 + exp64(-yd));
    y[d] = (float)yd;
  }
}

// Per-item constants of the FP64 sampler (up to 16 components), one row per
// wave in LDS: mu (80), 1/sigma (80), sigma (80), log pi_k - sum_d log
// sigma_kd - 5/2 log 2 pi (16), alpha.
constexpr int kMixMaxK = 16;
constexpr int kMixRowF64 = 16 * kMixMaxK + 1;

__device__ __forceinline__ void mix_prepare_f64(const uint32_t* thr, const float* mu, const float* sg, int K,
                                                double* row, int lane) {
  for (int i = lane; i < K * 5; i += kWave) {
    row[i] = (double)mu[i];
    row[80 + i] = 1.0 / (double)sg[i];
    row[160 + i] = (double)sg[i];
  }
  if (lane < K) {
    const double hi = lane + 1 < K ? (double)thr[lane + 1] : kTwo32;
    const double pk = (hi - (double)thr[lane]) / kTwo32;
    double c = -1e300;
    if (pk > 0.0) {
      c = log(pk) - 5.0 * kHalfLog2Pi;
      for (int d = 0; d < 5; ++d) c -= log((double)sg[lane * 5 + d]);
    }
    row[240 + lane] = c;
  }
  if (lane == 0) row[256] = (double)thr[0] / kTwo32;
}

// Draw u (and y = logit u) for one sample from the 8 words of two Philox blocks.
__device__ __forceinline__ void mix_draw_row_f64(const uint32_t x[8], const uint32_t* __restrict__ thr,
                                                 const double* row, int K, double u[5], double y[5]) {
  if (x[0] < thr[0]) {
    for (int d = 0; d < 5; ++d) {
      u[d] = unif23(x[1 + d] >> 9);
      y[d] = log64(u[d] * rcp64(1.0 - u[d]));
    }
    return;
  }
  int k = 0;
  for (int j = 1; j < K; ++j) k = x[0] >= thr[j] ? j : k;
  double z[6];
  for (int pr = 0; pr < 3; ++pr) {
    const double a1 = unif23(x[1 + 2 * pr] >> 9), a2 = unif23(x[2 + 2 * pr] >> 9);
    const double r = sqrt64(-2.0 * log64(a1));
    double sn, cs;
    sincos_2pi(a2, sn, cs);
    z[2 * pr] = r * cs;
    z[2 * pr + 1] = r * sn;
  }
  for (int d = 0; d < 5; ++d) {
    y[d] = row[k * 5 + d] + row[160 + k * 5 + d] * z[d];
    u[d] = rcp64(1.0 + exp64(-y[d]));
  }
}

// q(u) in FP64 from the row, the largest component scaled out; arguments
// below -800 (an exponential of 0) and above 1000 (inf) are clamped, as
// exp64 takes finite powers of two.
__device__ __forceinline__ double mix_density_f64(const double* row, int K, const double y[5]) {
  double mx = -1e300;
  for (int k = 0; k < K; ++k) {
    double l = row[240 + k];
    for (int d = 0; d < 5; ++d) {
      const double z = (y[d] - row[k * 5 + d]) * row[80 + k * 5 + d];
      l = fma(-0.5 * z, z, l);
    }
    mx = fmax(mx, l);
  }
  double acc = 0.0;
  for (int k = 0; k < K; ++k) {
    double l = row[240 + k];
    for (int d = 0; d < 5; ++d) {
      const double z = (y[d] - row[k * 5 + d]) * row[80 + k * 5 + d];
      l = fma(-0.5 * z, z, l);
    }
    acc += exp64(fmax(l - mx, -800.0));
  }
  double lq = mx + log64(acc);  // acc >= 1
  // log(u (1 - u)) = -|y| - 2 log(1 + e^-|y|); the five factors lie in [1, 2]
  double prod = 1.0;
  for (int d = 0; d < 5; ++d) {
    const double a = fabs(y[d]);
    lq += a;
    prod *= 1.0 + exp64(-fmin(a, 800.0));
  }
  lq += 2.0 * log64(prod);
  return row[256] + exp64(fmin(fmax(lq, -800.0), 1000.0));
}

__device__ __forceinline__ void mix_prepare_f32(const uint32_t* thr, const float* mu, const float* sg, int K,
                                                float* row, int lane) {
  for (int i = lane; i < K * 5; i += kWave) {
    row[i] = mu[i];
    row[40 + i] = (float)(rcp64((double)sg[i]) * 0.70710678118654752);
    row[kMixSigma + i] = sg[i];
  }
  // log pi_k - sum_d log sigma_kd - 5/2 log 2pi: the K x 6 logarithms one per
  // lane (lane 6k holds log pi_k, lanes 6k+1..6k+5 -log sigma_kd), gathered
  // by lane k; the wave waits for one logarithm instead of six in a row
  double lg = 0.0;
  const int kc = lane / 6, jc = lane - 6 * kc;
  if (lane < 6 * K) {
    if (jc == 0) {
      const double hi = kc + 1 < K ? (double)thr[kc + 1] : kTwo32;
      const double pk = (hi - (double)thr[kc]) * (1.0 / kTwo32);
      lg = pk > 0.0 ? log64(pk) : -1e30;
    } else {
      lg = -log64((double)sg[kc * 5 + jc - 1]);
    }
  }
  double c = -5.0 * kHalfLog2Pi;
#pragma unroll
  for (int t = 0; t < 6; ++t) c += __shfl(lg, min(6 * lane + t, kWave - 1), kWave);
  if (lane < K) row[80 + lane] = (float)c;
  if (lane == 0) row[88] = (float)((double)thr[0] / kTwo32);
}

// e^x and ln x from the hardware base-2 instructions (about one ulp; no
// special-case handling: the arguments here are finite, and a zero or
// subnormal sum of exponentials gives -inf or a large negative log, which
// leaves q = alpha through the final exponential)
__device__ __forceinline__ float exp_f32(float x) { return __builtin_amdgcn_exp2f(x * 1.4426950408889634f); }
__device__ __forceinline__ float log_f32(float x) { return __builtin_amdgcn_logf(x) * 0.6931471805599453f; }

__device__ __forceinline__ float mix_density_f32(const float* row, int K, const float yf[5]) {
  // l_k <= log pi_k - sum_d log sigma_kd - 5/2 log 2pi <= 35 (sigma >= e^-7), so the
  // exponentials need no max shift; all of them underflowing leaves q = alpha.
  // Unrolled over the 8 components the row holds, so the LDS reads of later
  // components are issued before the arithmetic of earlier ones waits.
  float acc = 0.f;
#pragma unroll
  for (int k = 0; k < kMixKF32; ++k) {
    if (k < K) {
      float l = row[80 + k];
#pragma unroll
      for (int d = 0; d < 5; ++d) {
        const float z = (yf[d] - row[k * 5 + d]) * row[40 + k * 5 + d];
        l = fmaf(-z, z, l);
      }
      acc += exp_f32(l);
    }
  }
  float lq = log_f32(acc);
  // log(u (1 - u)) = -|y| - 2 log(1 + e^-|y|); the five factors 1 + e^-|y|
  // lie in [1, 2], so their product takes one logarithm
  float prod = 1.0f;
#pragma unroll
  for (int d = 0; d < 5; ++d) {
    const float a = fabsf(yf[d]);
    lq += a;
    prod *= 1.0f + exp_f32(-a);
  }
  lq += 2.0f * log_f32(prod);
  return row[88] + exp_f32(lq);
}

// Set up the wave-uniform item constants.
// The item constants of a (cell, channel) pair: masses, threshold terms and
// the channel coefficient (the same for every observed node of the pair).
__device__ __forceinline__ void item_pair(Item& it, const CollideArgs& A, const Channel& ch, int cell) {
  const Grid& G = A.G;
  it.cell = cell;
  it.m1sq = A.mass2[ch.sp[0] * G.cells + cell];
  it.m2sq = A.mass2[ch.sp[1] * G.cells + cell];
  it.m3sq = A.mass2[ch.sp[2] * G.cells + cell];
  it.m4sq = A.mass2[ch.sp[3] * G.cells + cell];
  it.mu = A.mass2[kGluon * G.cells + cell];
  const double m3 = sqrt(it.m3sq), m4 = sqrt(it.m4sq);
  it.sum2 = (m3 + m4) * (m3 + m4);
  it.dif2 = (m3 - m4) * (m3 - m4);
  it.dm34 = it.m3sq - it.m4sq;
  it.dde = (it.m1sq - it.m2sq) - it.dm34;
  it.sde = (it.m1sq - it.m2sq) + it.dm34;
  const double V5 = G.Vp * 4.0 * kPi;
  it.coef = (A.symmetric ? ch.w : ch.sigma) * V5 / (double)A.n_samples;
}

// The observed node's part of the item constants (p1, E1, f1, prefactor).
__device__ __forceinline__ void item_node(Item& it, const CollideArgs& A, const Channel& ch, int p1_lin) {
  const Grid& G = A.G;
  it.p1_lin = p1_lin;
  const int iz = p1_lin % G.np[2];
  const int iy = (p1_lin / G.np[2]) % G.np[1];
  const int ix = p1_lin / (G.np[2] * G.np[1]);
  it.p1[0] = node_coord(G.ph[0], G.dp[0], ix);
  it.p1[1] = node_coord(G.ph[1], G.dp[1], iy);
  it.p1[2] = node_coord(G.ph[2], G.dp[2], iz);
  it.E1 = sqrt(it.p1[0] * it.p1[0] + it.p1[1] * it.p1[1] + it.p1[2] * it.p1[2] + it.m1sq);
  it.f1 = A.f64[((size_t)ch.sp[0] * G.cells + it.cell) * G.nodes + p1_lin];
  it.pref = it.coef * G.g4 * kNorm / it.E1;
}

__device__ __forceinline__ void load_item(Item& it, const CollideArgs& A, const Channel& ch, int cell, int p1_lin) {
  item_pair(it, A, ch, cell);
  item_node(it, A, ch, p1_lin);
}


// Per-sample value without the bracket, in precision R: |M|^2 times the
// phase-space prefactor.
template <typename R>
__device__ __forceinline__ R prefactor(const Item& it, const Geo& g) {
  return (R)it.pref * (R)g.pstar * (R)g.rs * rcp_r<R>((R)g.E2);
}

template <typename R, bool kUser = true>
__device__ __forceinline__ R weight_no_bracket(const CollideArgs& A, const Item& it, const Geo& g, int row) {
  const R m = msq_row<R, kUser>(A.msq_mask, A.msq, row, (R)g.s, (R)g.t, (R)g.u, (R)it.mu);
  return m * prefactor<R>(it, g);
}

__device__ __forceinline__ bool is_gluon(int sp) { return sp == kGluon; }

// Unbiased estimate of the variance of an item's direct sum S = sum_s v_s
// over N samples: N/(N-1) (sum v^2 - S^2/N).
__device__ __forceinline__ double item_variance(double s, double sq, int n) {
  if (n < 2) return 0.0;
  return fmax(0.0, (sq - s * s / n) * ((double)n / (n - 1)));
}

}  // namespace
}  // namespace qgbe
