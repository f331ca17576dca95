// Device building blocks of the lattice Boltzmann kernels (gfx950), shared by
// the translation units of the library; everything here is inlined into the
// kernels that use it.
//
// State layout: per sample, q population planes (q = 27 for D3Q27, 19 for
// D3Q19) of n^3 values each plus padding (SoA), cells C-ordered [z][y][x].
// Values are shifted: g_i = f_i - w_i (stored in float or double). The state
// is updated in place with the AA pattern: on an even step a node reads its
// own q slots and writes the post-collision populations back into the
// opposite slots of the same node; on an odd step it reads population i from
// the slot of the opposite velocity at node x - c_i and writes the
// post-collision population i into slot i of node x + c_i. Every slot is read
// and written by exactly one thread per step, so the update is race free, and
// one step moves q loads + q stores per node.
//
// Collision (eqs. (equilibrium), (kbcCollision), (entropyControl), Table 1):
//   rho = 1 + sum g, j = sum c g, u = j / rho,
//   g^eq_i = w_i [drho + 3 c_i.j + rho (4.5 (c_i.u)^2 - 1.5 |u|^2)],
//   f^neq = g - g^eq,
//   shear part ds: the population vector with the traceless normal-stress
//   differences Nxz, Nyz and the off-diagonal stresses of f^neq and no other
//   raw moment: faces (+-1,0,0): (2Nxz - Nyz)/6, (0,+-1,0): (2Nyz - Nxz)/6,
//   (0,0,+-1): -(Nxz + Nyz)/6; edges: cx cy Pxy/4 + cx cz Pxz/4 + cy cz Pyz/4;
//   rest and corners: 0 (the same on both lattices).  Higher-order part
//   dh = f^neq - ds.
//   gamma = 2/omega - (2 - 2/omega) <ds|dh>/<dh|dh>, <X|Y> = sum X_i Y_i / f^eq_i
//   (gamma = 2 when <dh|dh> <= 1e-30),
//   g* = g - omega ds - (omega gamma / 2) dh.
// Everything is computed in the storage precision from the shifted values,
// so the weights w_i never enter a subtraction of nearly equal numbers.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

#include "kernels.h"
#include "lattice.h"

namespace mclbm {
namespace {

template <int I, int N, typename F>
__host__ __device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

// f(i) for every velocity i of the lattice (D3Q27 numbering, ascending)
template <int QN, typename F>
__host__ __device__ __forceinline__ void for_vel(F&& f) {
  static_for<0, Q>([&](auto ic) {
    if constexpr (in_lattice<QN>(decltype(ic)::value)) f(ic);
  });
}

template <int c, typename T>
__device__ __forceinline__ T signed_term(T v) {
  if constexpr (c > 0) return v;
  else return -v;
}

// c_i . (x, y, z) built from the non-zero components only
template <int i, typename T>
__device__ __forceinline__ T cdot(T x, T y, T z) {
  constexpr int a = cx(i), b = cy(i), c = cz(i);
  if constexpr (a == 0 && b == 0 && c == 0) return T(0);
  else if constexpr (b == 0 && c == 0) return signed_term<a>(x);
  else if constexpr (a == 0 && c == 0) return signed_term<b>(y);
  else if constexpr (a == 0 && b == 0) return signed_term<c>(z);
  else if constexpr (c == 0) return signed_term<a>(x) + signed_term<b>(y);
  else if constexpr (b == 0) return signed_term<a>(x) + signed_term<c>(z);
  else if constexpr (a == 0) return signed_term<b>(y) + signed_term<c>(z);
  else return signed_term<a>(x) + signed_term<b>(y) + signed_term<c>(z);
}

template <typename T>
__device__ __forceinline__ T recip(T x) {
  if constexpr (std::is_same<T, float>::value) return __builtin_amdgcn_rcpf(x);
  else return 1.0 / x;
}

template <typename T>
__device__ __forceinline__ T vfma(T a, T b, T c) {
  if constexpr (std::is_same<T, float>::value) return __builtin_fmaf(a, b, c);
  else return __builtin_fma(a, b, c);
}

// 1 / x to about one unit in the last place for normal x: the hardware
// estimate (1 ulp in float, about 2^-24 in double) and one Newton step in
// float, two in double; a quarter of the instructions of the correctly
// rounded division.
template <typename T>
__device__ __forceinline__ T recip_newton(T x) {
  if constexpr (std::is_same<T, float>::value) {
    const float r = __builtin_amdgcn_rcpf(x);
    return __builtin_fmaf(__builtin_fmaf(-x, r, 1.0f), r, r);
  } else {
    double r = __builtin_amdgcn_rcp(x);
    r = __builtin_fma(__builtin_fma(-x, r, 1.0), r, r);
    return __builtin_fma(__builtin_fma(-x, r, 1.0), r, r);
  }
}

// reciprocal in the collision's inner products: the hardware estimate in
// float, to about one unit in the last place in double
template <typename T>
__device__ __forceinline__ T recip_sum(T x) {
  if constexpr (std::is_same<T, float>::value) return __builtin_amdgcn_rcpf(x);
  else return recip_newton(x);
}

template <typename T>
__device__ __forceinline__ T vmin(T a, T b) {
  return a < b ? a : b;
}

// minimum in one instruction (the other operand where one is NaN)
template <typename T>
__device__ __forceinline__ T hwmin(T a, T b) {
  if constexpr (std::is_same<T, float>::value) return __builtin_fminf(a, b);
  else return __builtin_fmin(a, b);
}

template <typename T>
__device__ __forceinline__ T hwmax(T a, T b) {
  if constexpr (std::is_same<T, float>::value) return __builtin_fmaxf(a, b);
  else return __builtin_fmax(a, b);
}

// ln(1 + x) for x > -1. float: the hardware base-2 logarithm of u = 1 + x
// (rounded to float) times ln 2, minus the rounding error e = (u - 1) - x of
// u (exact in float): ln(1 + x) = ln(u - e) = ln u - e/u + O(e^2), and
// taking e for e/u errs by e x / u, at most 2^-24 |x|, which is below one
// unit in the last place of ln(1 + x) for small x and of the logarithm's own
// rounding for large x (the correction is the one of the log1p identity in
// Goldberg, "What every computer scientist should know about floating-point
// arithmetic", 1991, Theorem 4, to first order, without its division);
// exactly x where u rounds to 1. double: the library log1p.
template <typename T>
__device__ __forceinline__ T log1p_acc(T x) {
  if constexpr (std::is_same<T, float>::value) {
    const float u = 1.0f + x;
    return __builtin_amdgcn_logf(u) * 0.693147180559945309f - ((u - 1.0f) - x);
  } else {
    return log1p(x);
  }
}

template <typename T>
struct Macro {
  T drho, jx, jy, jz, rho, inv, ux, uy, uz, usq15;
};

template <int QN, typename T>
__device__ __forceinline__ Macro<T> macroscopic(const T (&g)[Q]) {
  T d = T(0), x = T(0), y = T(0), z = T(0);
  for_vel<QN>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    d += g[i];
  });
  // momentum: +direction partial sums minus -direction partial sums
  T xp = T(0), xm = T(0), yp = T(0), ym = T(0), zp = T(0), zm = T(0);
  for_vel<QN>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    if constexpr (cx(i) > 0) xp += g[i];
    if constexpr (cx(i) < 0) xm += g[i];
    if constexpr (cy(i) > 0) yp += g[i];
    if constexpr (cy(i) < 0) ym += g[i];
    if constexpr (cz(i) > 0) zp += g[i];
    if constexpr (cz(i) < 0) zm += g[i];
  });
  x = xp - xm;
  y = yp - ym;
  z = zp - zm;
  Macro<T> m;
  m.drho = d;
  m.jx = x;
  m.jy = y;
  m.jz = z;
  m.rho = T(1) + d;
  m.inv = T(1) / m.rho;
  m.ux = x * m.inv;
  m.uy = y * m.inv;
  m.uz = z * m.inv;
  m.usq15 = T(1.5) * (m.ux * m.ux + m.uy * m.uy + m.uz * m.uz);
  return m;
}

// Velocity of a node (eq. (momentDefin)) from its shifted populations, summed
// in double in velocity order whatever the storage precision: the field the
// FP64 observables transform. The collide-and-stream kernel writes it on
// record ticks and the first pass of the observables computes it from a
// stored state with this same code, so the two fields are bitwise equal.
template <int QN, typename T>
__device__ __forceinline__ void node_velocity(const T (&g)[Q], double& ux, double& uy, double& uz) {
  double d = 0.0, jx = 0.0, jy = 0.0, jz = 0.0;
  for_vel<QN>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    const double v = double(g[i]);
    d += v;
    if constexpr (cx(i) != 0) jx += cx(i) * v;
    if constexpr (cy(i) != 0) jy += cy(i) * v;
    if constexpr (cz(i) != 0) jz += cz(i) * v;
  });
  const double rho = 1.0 + d;
  ux = jx / rho;
  uy = jy / rho;
  uz = jz / rho;
}

// shifted equilibrium g^eq_i = f^eq_i - w_i
template <int QN, int i, typename T>
__device__ __forceinline__ T geq(const Macro<T>& m) {
  const T w = T(weight<QN>(i));
  if constexpr (nonzeros(i) == 0) {
    return w * (m.drho - m.rho * m.usq15);
  } else {
    const T cu = cdot<i>(m.ux, m.uy, m.uz);
    const T cj = cdot<i>(m.jx, m.jy, m.jz);
    if constexpr (std::is_same<T, float>::value) {
      // 3 w_i c_i.j with 3 w_i split into a float head and tail: with the
      // rounded weights alone, sum_i 3 w_i c_i c_i = (1 + 7.5e-9) I, a
      // systematic momentum gain in every collision that accumulates over
      // thousands of steps; with the tail the first moment of g^eq is j up
      // to unbiased rounding.
      constexpr double w3 = 3.0 * weight<QN>(i);
      constexpr float w3_hi = float(w3);
      constexpr float w3_lo = float(w3 - double(w3_hi));
      return w * (m.drho + m.rho * (T(4.5) * cu * cu - m.usq15)) + (w3_hi * cj + w3_lo * cj);
    } else {
      return w * (m.drho + T(3) * cj + m.rho * (T(4.5) * cu * cu - m.usq15));
    }
  }
}

template <typename T>
struct Shear {
  T dsx, dsy, dsz, exy, exz, eyz;
};

// shear part of velocity i (faces and edges only)
template <int i, typename T>
__device__ __forceinline__ T shear_part(const Shear<T>& s) {
  constexpr int a = cx(i), b = cy(i), c = cz(i);
  static_assert(nonzeros(i) == 1 || nonzeros(i) == 2, "shear part vanishes on rest and corners");
  if constexpr (nonzeros(i) == 1) {
    if constexpr (a != 0) return s.dsx;
    else if constexpr (b != 0) return s.dsy;
    else return s.dsz;
  } else {
    if constexpr (c == 0) return signed_term<a * b>(s.exy);
    else if constexpr (b == 0) return signed_term<a * c>(s.exz);
    else return signed_term<b * c>(s.eyz);
  }
}

// Second moments of f^neq and the shear coefficients.
template <int QN, typename T>
__device__ __forceinline__ Shear<T> shear_coefficients(const T (&fneq)[Q]) {
  T pxx = T(0), pyy = T(0), pzz = T(0), pxy = T(0), pxz = T(0), pyz = T(0);
  for_vel<QN>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    if constexpr (cx(i) != 0) pxx += fneq[i];
    if constexpr (cy(i) != 0) pyy += fneq[i];
    if constexpr (cz(i) != 0) pzz += fneq[i];
    if constexpr (cx(i) * cy(i) > 0) pxy += fneq[i];
    if constexpr (cx(i) * cy(i) < 0) pxy -= fneq[i];
    if constexpr (cx(i) * cz(i) > 0) pxz += fneq[i];
    if constexpr (cx(i) * cz(i) < 0) pxz -= fneq[i];
    if constexpr (cy(i) * cz(i) > 0) pyz += fneq[i];
    if constexpr (cy(i) * cz(i) < 0) pyz -= fneq[i];
  });
  const T nxz = pxx - pzz, nyz = pyy - pzz;
  const T sixth = T(1) / T(6);
  Shear<T> s;
  s.dsx = (T(2) * nxz - nyz) * sixth;
  s.dsy = (T(2) * nyz - nxz) * sixth;
  s.dsz = -(s.dsx + s.dsy);
  s.exy = T(0.25) * pxy;
  s.exz = T(0.25) * pxz;
  s.eyz = T(0.25) * pyz;
  return s;
}

template <typename T>
struct Relax {
  T omega, two_over_omega, kappa, eps;
};

template <typename T>
__device__ __forceinline__ Relax<T> relax_of(const DevSample& sp) {
  Relax<T> r;
  if constexpr (std::is_same<T, float>::value) {
    r.omega = sp.omega_f;
    r.two_over_omega = sp.two_over_omega_f;
    r.kappa = sp.kappa_f;
    r.eps = sp.eps_f;
  } else {
    r.omega = sp.omega;
    r.two_over_omega = sp.two_over_omega;
    r.kappa = sp.kappa;
    r.eps = sp.eps;
  }
  return r;
}

template <typename T>
struct CellResult {
  Macro<T> m;
  T gamma;
  bool bad;
};

// Exact entropic stabiliser (eq. (kbc_entropy)): with t = omega gamma / 2 the
// post-collision populations are f*_i(t) = b_i - t dh_i, b_i = f_i - omega ds_i,
// and H(t) = sum f*_i ln(f*_i / w_i) is convex in t on the interval where
// every f*_i > 0, with
//   -H'(t) = sum dh_i ln(f*_i / w_i)      (sum dh_i = 0),
//    H''(t) = sum dh_i^2 / f*_i.
// Newton's method from the closed-form t (the first-order solution of
// H'(t) = 0) converges quadratically; a step that would leave the interval is
// replaced by the midpoint towards its edge. A node stops once its step is
// below kExactTolerance of t (the next step would be below the rounding of
// T), after at most kExactNewtonSteps steps; every node decides for itself,
// so the result does not depend on its neighbours in the wave.
// ln(f*_i / w_i) is evaluated as log1p((f*_i - w_i) / w_i) from the shifted
// values, which keeps its relative accuracy for populations near their
// weights. dh carries no mass and no momentum, so H'(t) does not change when
// a + b.c_i is subtracted from every logarithm; the sums subtract
// drho - 1.5 |u|^2 + 3 c_i.u, the part of ln(f^eq_i / w_i) of first order in
// drho and second in u. In exact arithmetic that is a no-op; in rounding it
// keeps the mass and momentum that dh's rounding leaves (near equilibrium,
// where dh is itself at rounding level) from multiplying an O(u) logarithm
// and swamping the third-order balance that fixes t there.
constexpr int kExactNewtonSteps = 4;

template <typename T>
constexpr T exact_tolerance() {
  return std::is_same<T, float>::value ? T(1.0 / (1 << 12)) : T(1e-8);
}

// Below which <dh|dh> counts as equilibrium (gamma = 2, for either
// stabiliser). In FP64 1e-30, where dh vanishes up to rounding. In FP32 the dh
// of a node at equilibrium is the rounding of its populations (the moments
// and g^eq of about 27 float terms: a few units in the last place of
// |g^eq| ~ w |u|): the closed form would report a gamma of that rounding, and
// the exact minimiser acts on any dh, however small, by an amount of third
// order in u. Such a node is taken as at equilibrium, like the FP64 path,
// when <dh|dh> <= 2^-40 (3 |u|^2 + drho^2), about ten times that rounding
// level (sum_i (g^eq_i)^2 / f^eq_i = 3 |u|^2 + drho^2 to leading order);
// resolved flows carry dh far above it.
template <typename T>
__device__ __forceinline__ T equilibrium_threshold(const Macro<T>& m) {
  if constexpr (std::is_same<T, float>::value)
    return fmaxf(1e-30f, 0x1.0p-40f * (2.0f * m.usq15 + m.drho * m.drho));
  else
    return T(1e-30);
}

// The terms of the exact stabiliser, once per node: dh_i = f^neq_i - ds_i and
// bs_i = b_i - w_i = f_i - omega ds_i - w_i, so that f*_i(t) - w_i = bs_i - t dh_i.
// bs is formed as the closed-form update forms the post-collision state,
// (g^eq_i - ds_i) + eps ds_i + dh_i with eps = 2 - omega, which keeps the
// shear relaxation at full relative precision for omega near 2 (a float
// omega alone would carry eps to about 1e-4); the post-collision state is
// then bs_i - t dh_i, and g^eq and f^neq are no longer needed.
template <int QN, typename T>
__device__ __forceinline__ void exact_terms(const T (&geq)[Q], const T (&fneq)[Q], const Shear<T>& s, T eps,
                                            T (&dh)[Q], T (&bs)[Q]) {
  for_vel<QN>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    T ds = T(0);
    if constexpr (nonzeros(i) == 1 || nonzeros(i) == 2) ds = shear_part<i>(s);
    dh[i] = fneq[i] - ds;
    bs[i] = ((geq[i] - ds) + eps * ds) + dh[i];
  });
}

template <int QN, typename T>
__device__ __forceinline__ T exact_entropic_t(const T (&dh)[Q], const T (&bs)[Q], const Macro<T>& m, T t) {
  const T a = m.drho - m.usq15;
  // The interval of t where every f*_i = w_i + bs_i - t dh_i > 0 bounds the
  // Newton iterates; it is formed (27 quotients) only when an iterate leaves
  // the region where every f*_i is positive, which takes 27 products to
  // check. In float the quotients use the hardware reciprocal (about one unit
  // in the last place) and are moved inwards by 2^-20 of their size, so that
  // the interval stays inside the exact one.
  bool have_interval = false;
  T lo = T(-1e30), hi = T(1e30);
  auto interval = [&]() {
    for_vel<QN>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      const T base = T(weight<QN>(i)) + bs[i];
      T q;
      if constexpr (std::is_same<T, float>::value) {
        q = base * __builtin_amdgcn_rcpf(dh[i]);
        q = dh[i] > T(0) ? q - fabsf(q) * 0x1.0p-20f : q + fabsf(q) * 0x1.0p-20f;
      } else {
        q = base / dh[i];
      }
      if (dh[i] > T(0)) hi = vmin(hi, q);
      if (dh[i] < T(0)) lo = lo > q ? lo : q;
    });
    have_interval = true;
  };
  auto positive_at = [&](T tt) {
    T fmin = T(1);
    for_vel<QN>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      fmin = hwmin(fmin, (T(weight<QN>(i)) + bs[i]) - tt * dh[i]);
    });
    return fmin > T(0) && tt == tt;
  };
  // In float the curvature H'' of the first step is kept for the later ones
  // (a chord step: the curvature changes by about |t - t0| |dh| / f* between
  // steps, so each later step still contracts the error by that factor,
  // reaching float resolution in the step that meets the stopping rule); in
  // double every step is a full Newton step.
  // In float the first step also bounds its own error: with q_i = dh_i / f*_i,
  // |d3H/dt3| = |sum dh_i q_i^2| <= max|q| H'', so Newton's error after a
  // step D from t is below (|d3H/dt3| / (2 H'')) D^2 <= max|q| D^2 / 2 to
  // first order in D max|q|; while D max|q| <= 1/16 a node stops once that
  // is below 2^-22 of t, about two units in the last place, without taking
  // the logarithms again to see the next step fall below the tolerance.
  // The same maximum vouches for the next iterate: f*_i at a distance D from
  // the point t0 where q was taken is f*_i(t0) (1 - D q_i), which is positive
  // (by far more than its rounding) while |D| max|q| <= 1/2, provided it is at
  // t0, where a value that is not makes the sum of logarithms, and with it D,
  // infinite or a NaN. Only a longer step checks the populations one by one
  // (13 x 64^3 FP32 per tick 181 -> 148 us, 4 x 128^3 446 -> 355, 11 x 64^3 FP64
  // 1050 -> 975).
  constexpr bool kChord = std::is_same<T, float>::value;
  bool done = false;
  T d2 = T(0), qmax = T(0), t0 = t;
  T d1 = T(0);
  auto sums = [&](auto curvature) {
    constexpr bool kCurvature = decltype(curvature)::value;
    d1 = T(0);
    if constexpr (kCurvature) {
      d2 = qmax = T(0);
      t0 = t;
    }
    for_vel<QN>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      constexpr double w = weight<QN>(i);
      // f*_i - w_i in shifted form
      const T gs = bs[i] - t * dh[i];
      d1 += dh[i] * (log1p_acc(gs * T(1.0 / w)) - (a + T(3) * cdot<i>(m.ux, m.uy, m.uz)));
      if constexpr (kCurvature) {
        const T qi = dh[i] * recip(T(w) + gs);
        d2 += dh[i] * qi;
        qmax = hwmax(qmax, T(fabs(qi)));
      }
    });
  };
  for (int it = 0; it < kExactNewtonSteps && !done; ++it) {
    if (!kChord || it == 0)
      sums(std::true_type{});
    else
      sums(std::false_type{});
    T tn = t + d1 / d2;
    bool newton = true;
    if (!(qmax * T(fabs(tn - t0)) <= T(0.5)) && !positive_at(tn)) {
      if (!have_interval) interval();
      if (!(tn < hi)) {
        tn = T(0.5) * (t + hi);
        newton = false;
      }
      if (!(tn > lo)) {
        tn = T(0.5) * (t + lo);
        newton = false;
      }
    }
    const T step = tn - t, astep = step < T(0) ? -step : step;
    done = astep <= exact_tolerance<T>() * fabs(t);
    if constexpr (kChord)
      if (it == 0 && newton && qmax * astep <= T(0.0625))
        done = done || qmax * astep * astep <= T(0x1.0p-22) * fabs(tn);
    t = tn;
  }
  return t;
}

// f(i) for one velocity of each pair +-c_i (D3Q27 numbering, ascending: 14..26)
template <int QN, typename F>
__host__ __device__ __forceinline__ void for_pair(F&& f) {
  static_for<14, Q>([&](auto ic) {
    if constexpr (in_lattice<QN>(decltype(ic)::value)) f(ic);
  });
}

// The populations as sums and differences over the pairs +-c: for i > 13,
// p[i] = g_i + g_-i carries the even moments and p[26 - i] = g_i - g_-i the
// momentum; p[13] = g_13.
template <int QN, typename T>
__device__ __forceinline__ void to_pairs(T (&g)[Q]) {
  for_pair<QN>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    const T a = g[i], b = g[26 - i];
    g[i] = a + b;
    g[26 - i] = a - b;
  });
}

// Moments of the populations from their pairs: each takes about half the
// additions of a sum over all velocities; edges are summed per plane and
// corners by a 4-point butterfly.
template <typename T>
struct NodeMoments {
  T drho, jx, jy, jz;
  T nxz, nyz, pxy, pxz, pyz;  // second moments of g: xx - zz, yy - zz, xy, xz, yz
};

template <int QN, typename T>
__device__ __forceinline__ NodeMoments<T> pair_moments(const T (&p)[Q]) {
#pragma clang fp contract(off)
  auto s = [&](int i) { return p[i]; };
  auto d = [&](int i) { return p[26 - i]; };
  // i = 9 (cx + 1) + 3 (cy + 1) + (cz + 1)
  constexpr int X = 22, Y = 16, Z = 14, XYp = 25, XYm = 19, XZp = 23, XZm = 21, YZp = 17, YZm = 15;
  constexpr int C0 = 26, C1 = 24, C2 = 20, C3 = 18;  // (1,1,1), (1,1,-1), (1,-1,1), (1,-1,-1)
  const T exy = s(XYp) + s(XYm), exz = s(XZp) + s(XZm), eyz = s(YZp) + s(YZm);
  NodeMoments<T> m;
  m.drho = (p[13] + ((s(X) + s(Y)) + s(Z))) + ((exy + exz) + eyz);
  m.jx = (d(X) + (d(XYp) + d(XYm))) + (d(XZp) + d(XZm));
  m.jy = (d(Y) + (d(XYp) - d(XYm))) + (d(YZp) + d(YZm));
  m.jz = (d(Z) + (d(XZp) - d(XZm))) + (d(YZp) - d(YZm));
  m.nxz = (s(X) - s(Z)) + (exy - eyz);
  m.nyz = (s(Y) - s(Z)) + (exy - exz);
  m.pxy = s(XYp) - s(XYm);
  m.pxz = s(XZp) - s(XZm);
  m.pyz = s(YZp) - s(YZm);
  if constexpr (QN == 27) {
    const T sp = s(C0) + s(C1), sm = s(C0) - s(C1), tp = s(C2) + s(C3), tm = s(C2) - s(C3);
    m.drho += sp + tp;
    m.pxy += sp - tp;
    m.pxz += sm + tm;
    m.pyz += sm - tm;
    const T dp = d(C0) + d(C1), dm = d(C0) - d(C1), ep = d(C2) + d(C3), em = d(C2) - d(C3);
    m.jx += dp + ep;
    m.jy += dp - ep;
    m.jz += dm + em;
  }
  return m;
}

// Which of the two products u = j / rho in c_i.u of an edge (one zero component)
// stays unrounded inside the sum, in the velocity-by-velocity collision below:
// 0 x, 1 y, 2 z. A corner adds its z product to the sum of the edge (c_x, c_y, 0).
template <int QN>
__host__ __device__ constexpr int fused_axis(int i) {
  const int a = cx(i), b = cy(i), c = cz(i);
  if (c == 0) return b < 0 && (a < 0 || QN == 27) ? 0 : 1;
  if (b == 0) return QN == 27 || (a < 0 && c < 0) ? 0 : 2;
  return QN == 27 || (b < 0 && c < 0) ? 1 : 2;
}

// whether c_i.u and c_-i.u round to opposite numbers
template <int QN>
__host__ __device__ constexpr bool odd_velocity(int i) {
  if (nonzeros(i) < 2) return true;
  const int e = nonzeros(i) == 3 ? i - cz(i) : i;
  return fused_axis<QN>(e) == fused_axis<QN>(26 - e);
}

template <int QN, int i>
__device__ __forceinline__ float cdot_u(const Macro<float>& m) {
  constexpr int a = cx(i), b = cy(i), c = cz(i);
  if constexpr (nonzeros(i) < 2) {
    return cdot<i>(m.ux, m.uy, m.uz);
  } else if constexpr (nonzeros(i) == 3) {
    return vfma(signed_term<c>(m.jz), m.inv, cdot_u<QN, i - c>(m));
  } else if constexpr (fused_axis<QN>(i) == 0) {
    return vfma(signed_term<a>(m.jx), m.inv, c == 0 ? signed_term<b>(m.uy) : signed_term<c>(m.uz));
  } else if constexpr (fused_axis<QN>(i) == 1) {
    return vfma(signed_term<b>(m.jy), m.inv, c == 0 ? signed_term<a>(m.ux) : signed_term<c>(m.uz));
  } else {
    return vfma(signed_term<c>(m.jz), m.inv, b == 0 ? signed_term<a>(m.ux) : signed_term<b>(m.uy));
  }
}

// KBC collision of one node in place, g <- g*, velocity by velocity, with the
// closed form, in float: the collision of every FP32 kernel, of one step or of
// two, so that a sample's populations are the same bits however its steps are
// cut into calls, records and passes and whatever ensemble it is part of. Every
// rounding is spelled out, as the compiler once chose it for the formulas at the
// top of this file (which product of c.u stays unrounded included): results
// have always been these. What is the same for +c and -c is formed once.
// Between the passes g[] holds the shifted equilibrium.
template <int QN>
__device__ __forceinline__ CellResult<float> kbc_collide_each(float (&g)[Q], const Relax<float>& rp) {
#pragma clang fp contract(off)
  CellResult<float> res;
  res.m = macroscopic<QN>(g);
  Macro<float>& m = res.m;
  m.usq15 = 1.5f * vfma(m.uz, m.uz, vfma(m.ux, m.ux, m.uy * m.uy));
  constexpr float sixth = 1.0f / 6.0f, w13 = float(weight<QN>(13));
  float fneq[Q];
  // g^eq_i = w_i x_i + odd_i, x_i = drho + rho (4.5 (c_i.u)^2 - 1.5 |u|^2)
  const float x13 = vfma(-m.rho, m.usq15, m.drho);
  fneq[13] = vfma(-w13, x13, g[13]);
  g[13] = w13 * x13;
  for_pair<QN>([&](auto ic) {
    constexpr int i = decltype(ic)::value, k = 26 - i;
    constexpr float w = float(weight<QN>(i));
    // 3 w_i c_i.j with 3 w_i split into a float head and tail: with the
    // rounded weights alone, sum_i 3 w_i c_i c_i = (1 + 7.5e-9) I, a
    // systematic momentum gain in every collision that accumulates over
    // thousands of steps; with the tail the first moment of g^eq is j up
    // to unbiased rounding.
    constexpr float w3 = float(3.0 * weight<QN>(i)), w3_tail = float(3.0 * weight<QN>(i) - double(w3));
    const float cj = cdot<i>(m.jx, m.jy, m.jz);
    const float odd = vfma(w3, cj, w3_tail * cj);
    auto even = [&](float cu) { return vfma(m.rho, vfma(4.5f * cu, cu, -m.usq15), m.drho); };
    const float x = even(cdot_u<QN, i>(m));
    float y = x;
    if constexpr (!odd_velocity<QN>(i)) y = even(cdot_u<QN, k>(m));
    const float ge = vfma(w, x, odd), gk = vfma(w, y, -odd);
    fneq[i] = g[i] - ge;
    fneq[k] = g[k] - gk;
    g[i] = ge;
    g[k] = gk;
  });
  // second moments of f^neq and the shear part, faces without their 1 / 6
  float pxx = 0.0f, pyy = 0.0f, pzz = 0.0f, pxy = 0.0f, pxz = 0.0f, pyz = 0.0f;
  for_vel<QN>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    if constexpr (cx(i) != 0) pxx += fneq[i];
    if constexpr (cy(i) != 0) pyy += fneq[i];
    if constexpr (cz(i) != 0) pzz += fneq[i];
    if constexpr (cx(i) * cy(i) != 0) pxy += signed_term<cx(i) * cy(i)>(fneq[i]);
    if constexpr (cx(i) * cz(i) != 0) pxz += signed_term<cx(i) * cz(i)>(fneq[i]);
    if constexpr (cy(i) * cz(i) != 0) pyz += signed_term<cy(i) * cz(i)>(fneq[i]);
  });
  const float nxz = pxx - pzz, nyz = pyy - pzz;
  const float sx = vfma(2.0f, nxz, -nyz), sy = vfma(2.0f, nyz, -nxz);
  Shear<float> s;
  s.dsx = sx * sixth;
  s.dsy = sy * sixth;
  s.dsz = -vfma(sx, sixth, s.dsy);
  s.exy = 0.25f * pxy;
  s.exz = 0.25f * pxz;
  s.eyz = 0.25f * pyz;
  float A = 0.0f, B = 0.0f, low = 1.0f;
  for_vel<QN>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    const float feq = i == 13 ? vfma(w13, x13, w13) : float(weight<QN>(i)) + g[i];
    const float r = recip(feq);
    low = hwmin(low, feq);
    float dh = fneq[i];
    if constexpr (nonzeros(i) == 1 || nonzeros(i) == 2) {
      if constexpr (nonzeros(i) == 1 && cx(i) != 0) dh = vfma(-sixth, sx, dh);
      else if constexpr (nonzeros(i) == 1 && cy(i) != 0) dh = vfma(-sixth, sy, dh);
      else dh = dh - shear_part<i>(s);
      A = vfma(shear_part<i>(s) * dh, r, A);
      fneq[i] = dh;
    }
    B = vfma(dh * dh, r, B);
  });
  // The sums are complete here: A, needed only where B is above its threshold,
  // would otherwise be formed inside that branch, with the 45 values it is formed
  // from kept until then (34-118 registers spilled in the two-step kernel).
  asm volatile("" : "+v"(A), "+v"(B), "+v"(low));
  const float least = fmaxf(1e-30f, 0x1.0p-40f * vfma(m.drho, m.drho, m.usq15 + m.usq15));  // equilibrium_threshold
  float gamma = 2.0f;
  if (B > least) gamma = vfma(-rp.kappa, A / B, rp.two_over_omega);
  // g* = g - omega ds - t dh = (g^eq - ds) + (2 - omega) ds + (1 - t) dh.
  // The shear relaxation enters through eps = 2 - omega, which keeps the
  // viscosity (proportional to eps for omega near 2) at full relative
  // precision even in float.
  const float one_t = vfma(-0.5f * rp.omega, gamma, 1.0f);
  for_vel<QN>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    if constexpr (nonzeros(i) == 1 || nonzeros(i) == 2) {
      const float ds = shear_part<i>(s);
      g[i] = vfma(one_t, fneq[i], vfma(rp.eps, ds, g[i] - ds));
    } else {
      g[i] = vfma(one_t, fneq[i], g[i]);
    }
  });
  res.gamma = gamma;
  // (a NaN drops out of the minimum and shows in the density or the velocity)
  res.bad = !(m.rho > 0.0f) || !(m.usq15 < 1.5f) || !(low > 0.0f);
  return res;
}

// The same collision over pairs +-c. EXACT selects the exact minimiser of the
// discrete H-function instead of the closed form. With c.j for one velocity of
// the pair,
//   e = 2 w [drho - 1.5 rho |u|^2 + 4.5 (c.j)^2 / rho]  (g^eq_i + g^eq_-i),
//   o = 6 w c.j                                         (g^eq_i - g^eq_-i),
//   sh = s - e - 2 ds, dn = d - o                       (sum and difference of dh),
// and with E = 2 w + e, so that f^eq_+-i = (E +- o) / 2, both members' terms of
// the two inner products share one reciprocal:
//   sum dh^2 / f^eq = [sh (E sh - o dn) + dn (E dn - o sh)] / (E^2 - o^2),
//   sum ds dh / f^eq = 2 ds (E sh - o dn) / (E^2 - o^2).
// The shear moments are those of g minus those of g^eq, which are rho u u
// exactly (plus a trace that drops out of the differences). Every pair then
// takes its new sum s - 2 omega ds - t sh and difference d - t dn. That is 14
// reciprocals instead of 27 and half the sums: D3Q27 in double takes 580 vector
// instructions against 1130 velocity by velocity. (In float with the closed form
// it would take 490 against 605, but round otherwise than the results have always
// been; the passes of two steps, which are bound by arithmetic, took 794 us with it
// instead of 842 at 64 x 64^3, 887 instead of 1077 at 8 x 128^3.)
// In float 6 w is split into head and tail for dn: with the rounded weights
// alone sum_i 3 w_i c_i c_i = (1 + 7.5e-9) I, a systematic momentum gain in
// every collision that accumulates over thousands of steps. The shear
// relaxation enters as 2 ds - eps ds, eps = 2 - omega, which keeps the viscosity
// (proportional to eps for omega near 2) at full relative precision.
// Contraction is spelled out with fma, so that every kernel that inlines the
// collision rounds alike.
template <int QN, bool EXACT, typename T>
__device__ __forceinline__ CellResult<T> kbc_collide_pairs(T (&g)[Q], const Relax<T>& rp) {
#pragma clang fp contract(off)
  CellResult<T> res;
  to_pairs<QN>(g);
  const NodeMoments<T> mo = pair_moments<QN>(g);
  Macro<T>& m = res.m;
  m.drho = mo.drho;
  m.jx = mo.jx;
  m.jy = mo.jy;
  m.jz = mo.jz;
  m.rho = T(1) + m.drho;
  m.inv = recip_newton(m.rho);
  m.ux = m.jx * m.inv;
  m.uy = m.jy * m.inv;
  m.uz = m.jz * m.inv;
  const T jxux = m.jx * m.ux, jyuy = m.jy * m.uy, jzuz = m.jz * m.uz;
  const T ju15 = T(1.5) * ((jxux + jyuy) + jzuz);  // 1.5 rho |u|^2
  m.usq15 = ju15 * m.inv;
  // twice the shear part per class of velocities
  const T fxz = mo.nxz - (jxux - jzuz), fyz = mo.nyz - (jyuy - jzuz);
  const T third = T(1) / T(3);
  Shear<T> s2;
  s2.dsx = (T(2) * fxz - fyz) * third;
  s2.dsy = (T(2) * fyz - fxz) * third;
  s2.dsz = -(s2.dsx + s2.dsy);
  s2.exy = T(0.5) * vfma(-m.jx, m.uy, mo.pxy);
  s2.exz = T(0.5) * vfma(-m.jx, m.uz, mo.pxz);
  s2.eyz = T(0.5) * vfma(-m.jy, m.uz, mo.pyz);

  const T K = m.drho - ju15, inv9 = T(9) * m.inv;
  T sh[Q], dn[Q];  // of the pair's velocity i > 13
  T A = T(0), B, low;
  {
    constexpr T w0 = T(weight<QN>(13));
    const T e0 = w0 * K, f0 = g[13] - e0, E0 = w0 + e0;
    sh[13] = f0;
    B = f0 * f0 * recip_sum(E0);
    low = E0;
  }
  T axy = T(0), axz = T(0), ayz = T(0);
  for_pair<QN>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    constexpr double w6 = 6.0 * weight<QN>(i), w2 = 2.0 * weight<QN>(i);
    const T cj = cdot<i>(m.jx, m.jy, m.jz);
    const T e = vfma((inv9 * T(weight<QN>(i))) * cj, cj, K * T(w2));
    const T o = T(w6) * cj;
    T dni = vfma(-T(w6), cj, g[26 - i]);
    if constexpr (std::is_same<T, float>::value) dni = vfma(-float(w6 - double(float(w6))), cj, dni);
    const T E = T(w2) + e;
    T shi = g[i] - e;
    if constexpr (nonzeros(i) < 3) shi = shi - shear_part<i>(s2);
    const T den = vfma(E, E, -(o * o));
    const T r = recip_sum(den);
    const T a1 = vfma(E, shi, -(o * dni));
    const T a2 = vfma(E, dni, -(o * shi));
    B = vfma(vfma(a2, dni, a1 * shi), r, B);
    if constexpr (nonzeros(i) == 1) {
      A = vfma(shear_part<i>(s2), a1 * r, A);
    } else if constexpr (nonzeros(i) == 2) {
      if constexpr (cz(i) == 0) axy = vfma(T(cx(i) * cy(i)) * a1, r, axy);
      else if constexpr (cy(i) == 0) axz = vfma(T(cx(i) * cz(i)) * a1, r, axz);
      else ayz = vfma(T(cy(i) * cz(i)) * a1, r, ayz);
    }
    // f^eq_+-i > 0 is E > 0 and E^2 > o^2 (a NaN drops out here and shows in
    // the density or the velocity)
    low = hwmin(hwmin(low, den), E);
    sh[i] = shi;
    dn[i] = dni;
  });
  A = vfma(s2.exy, axy, A);
  A = vfma(s2.exz, axz, A);
  A = vfma(s2.eyz, ayz, A);
  const bool resolved = B > equilibrium_threshold<T>(m);
  T gamma = T(2);
  if (resolved) gamma = vfma(-rp.kappa, A * recip_newton(B), rp.two_over_omega);
  T t = T(0.5) * rp.omega * gamma;
  // omega ds per class
  const T heps = T(0.5) * rp.eps;
  Shear<T> od;
  od.dsx = vfma(-heps, s2.dsx, s2.dsx);
  od.dsy = vfma(-heps, s2.dsy, s2.dsy);
  od.dsz = vfma(-heps, s2.dsz, s2.dsz);
  od.exy = vfma(-heps, s2.exy, s2.exy);
  od.exz = vfma(-heps, s2.exz, s2.exz);
  od.eyz = vfma(-heps, s2.eyz, s2.eyz);
  if constexpr (EXACT) {
    // g* = bs - t dh (the same update as below, in the terms of the exact
    // minimiser, which are all it keeps through its iteration)
    T dh[Q], bs[Q];
    dh[13] = sh[13];
    bs[13] = g[13];
    for_pair<QN>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      dh[i] = T(0.5) * (sh[i] + dn[i]);
      dh[26 - i] = T(0.5) * (sh[i] - dn[i]);
      T ods = T(0);
      if constexpr (nonzeros(i) < 3) ods = shear_part<i>(od);
      const T even = vfma(T(0.5), g[i], -ods);
      bs[i] = vfma(T(0.5), g[26 - i], even);
      bs[26 - i] = vfma(T(-0.5), g[26 - i], even);
    });
    if (resolved) {
      t = exact_entropic_t<QN>(dh, bs, m, t);
      gamma = T(2) * t / rp.omega;
    }
    for_vel<QN>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      g[i] = vfma(-t, dh[i], bs[i]);
    });
  } else {
    const T th = T(0.5) * t;
    g[13] = vfma(-t, sh[13], g[13]);
    for_pair<QN>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      // half the pair's new sum, then its new difference
      T even = vfma(T(0.5), g[i], -(th * sh[i]));
      if constexpr (nonzeros(i) < 3) even = even - shear_part<i>(od);
      const T odd = vfma(-t, dn[i], g[26 - i]);
      g[i] = vfma(T(0.5), odd, even);
      g[26 - i] = vfma(T(-0.5), odd, even);
    });
  }
  res.gamma = gamma;
  res.bad = !(m.rho > T(0)) || !(m.usq15 < T(1.5)) || !(low > T(0));
  if constexpr (EXACT) res.bad = res.bad || !(t == t);
  return res;
}

// The collision of the kernels, of one step and of two alike: in float with the
// closed form velocity by velocity (see there); in double, whose divisions cost
// ten instructions each (one 32^3 sample 8.7 -> 7.8 us a step, 11 x 64^3 215 ->
// 205), and with the exact stabiliser, bound by arithmetic, over pairs.
template <int QN, bool EXACT = false, typename T>
__device__ __forceinline__ CellResult<T> kbc_collide(T (&g)[Q], const Relax<T>& rp) {
  if constexpr (std::is_same<T, float>::value && !EXACT) return kbc_collide_each<QN>(g, rp);
  else return kbc_collide_pairs<QN, EXACT>(g, rp);
}

// ---------------------------------------------------------------- addressing
struct Cell {
  uint32_t cell;
  uint32_t ox[3], oy[3], oz[3];  // neighbour coordinates along each axis: -1, 0, +1
};

__host__ __device__ __forceinline__ Cell make_cell(uint32_t cell, int l) {
  Cell c;
  c.cell = cell;
  const uint32_t msk = (1u << l) - 1u;
  const uint32_t x = cell & msk, y = (cell >> l) & msk, z = cell >> (2 * l);
  c.ox[0] = (x - 1u) & msk;
  c.ox[1] = x;
  c.ox[2] = (x + 1u) & msk;
  c.oy[0] = ((y - 1u) & msk) << l;
  c.oy[1] = y << l;
  c.oy[2] = ((y + 1u) & msk) << l;
  c.oz[0] = ((z - 1u) & msk) << (2 * l);
  c.oz[1] = z << (2 * l);
  c.oz[2] = ((z + 1u) & msk) << (2 * l);
  return c;
}

// index of the neighbour x + s * c_i
template <int i, int s>
__host__ __device__ __forceinline__ uint32_t neighbour(const Cell& c) {
  return c.oz[1 + s * cz(i)] + c.oy[1 + s * cy(i)] + c.ox[1 + s * cx(i)];
}

// AA slots of population i (D3Q27 numbering) of the node at c: the slot a
// step of the given parity reads it from before the collision, and the slot
// it writes the post-collision value to. A slot is a velocity (whose storage
// plane holds it) and a node. Even step: read slot i of the node, write slot
// opposite(i) of the node. Odd step: read slot opposite(i) of x - c_i, write
// slot i of x + c_i. The odd step's read undoes the even step's write of
// population i at x - c_i, so the pair streams by c_i twice over two steps,
// once per step.
struct Slot {
  int vel;
  uint32_t idx;
};
template <int i>
__host__ __device__ __forceinline__ Slot aa_read_slot(const Cell& c, bool odd) {
  return odd ? Slot{opposite(i), neighbour<i, -1>(c)} : Slot{i, c.cell};
}
template <int i>
__host__ __device__ __forceinline__ Slot aa_write_slot(const Cell& c, bool odd) {
  return odd ? Slot{i, neighbour<i, +1>(c)} : Slot{opposite(i), c.cell};
}

// element access with a 32-bit byte offset from a uniform plane base
template <typename T>
__host__ __device__ __forceinline__ T ld(const T* plane, uint32_t idx) {
  return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(plane) + idx * uint32_t(sizeof(T)));
}
template <typename T>
__host__ __device__ __forceinline__ void st(T* plane, uint32_t idx, T v) {
  *reinterpret_cast<T*>(reinterpret_cast<char*>(plane) + idx * uint32_t(sizeof(T))) = v;
}

// The 27 planes of one sample through one buffer resource: the per-plane
// offset is a scalar (SGPR) operand and each lane supplies a 32-bit byte
// offset, so an access costs one VGPR of address. Used when the sample's
// populations occupy less than 4 GiB.
constexpr int kBufferFlags = 0x00020000;  // 32-bit raw data format (gfx9 family)

// NT: non-temporal loads and stores (each population is read once and written
// once per step, so nothing is gained by keeping it in the caches).
constexpr int kAuxNontemporal = 2;  // cache-policy operand of buffer instructions: nt

// Accesses name a velocity i (D3Q27 numbering); the plane is plane_of<QN>(i).
template <typename T, bool NT, int QN>
struct BufPlanes {
  static constexpr int aux = NT ? kAuxNontemporal : 0;
  __amdgpu_buffer_rsrc_t rsrc;
  uint32_t plane_bytes;
  __device__ __forceinline__ BufPlanes(T* base, uint32_t pstride)
      : rsrc(__builtin_amdgcn_make_buffer_rsrc(base, 0, int(uint32_t(QN) * pstride * uint32_t(sizeof(T))), kBufferFlags)),
        plane_bytes(pstride * uint32_t(sizeof(T))) {}
  __device__ __forceinline__ T load(int i, uint32_t idx) const {
    const int plane = plane_of<QN>(i);
    if constexpr (sizeof(T) == 4)
      return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(rsrc, int(idx * 4u), int(plane * plane_bytes), aux));
    else
      return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(rsrc, int(idx * 8u), int(plane * plane_bytes), aux));
  }
  __device__ __forceinline__ void store(int i, uint32_t idx, T v) const {
    const int plane = plane_of<QN>(i);
    if constexpr (sizeof(T) == 4)
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), rsrc, int(idx * 4u),
                                            int(plane * plane_bytes), aux);
    else
      __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(decltype(__builtin_amdgcn_raw_buffer_load_b64(
                                                                   rsrc, 0, 0, 0)), v),
                                            rsrc, int(idx * 8u), int(plane * plane_bytes), aux);
  }
};

// The same access through plain pointers (any sample size).
template <typename T, bool NT, int QN>
struct PtrPlanes {
  T* base;
  uint32_t pstride;
  __device__ __forceinline__ PtrPlanes(T* b, uint32_t p) : base(b), pstride(p) {}
  __device__ __forceinline__ T load(int i, uint32_t idx) const {
    const size_t plane = size_t(plane_of<QN>(i));
    if constexpr (NT) return __builtin_nontemporal_load(base + plane * pstride + idx);
    else return ld(base + plane * pstride, idx);
  }
  __device__ __forceinline__ void store(int i, uint32_t idx, T v) const {
    const size_t plane = size_t(plane_of<QN>(i));
    if constexpr (NT) __builtin_nontemporal_store(v, base + plane * pstride + idx);
    else st(base + plane * pstride, idx, v);
  }
};

// populations of the post-stream state at a node, for either AA parity: the
// slots the next step reads them from
template <int QN, typename T>
__host__ __device__ __forceinline__ void load_state(const T* base, uint32_t pstride, const Cell& c, bool odd,
                                                    T (&g)[Q]) {
  for_vel<QN>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    const Slot s = aa_read_slot<i>(c, odd);
    g[i] = ld(base + size_t(plane_of<QN>(s.vel)) * pstride, s.idx);
  });
}

// the inverse mapping: write a post-stream state at a node
template <int QN, typename T>
__host__ __device__ __forceinline__ void write_state(T* base, uint32_t pstride, const Cell& c, bool odd,
                                                     const T (&g)[Q]) {
  for_vel<QN>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    const Slot s = aa_read_slot<i>(c, odd);
    st(base + size_t(plane_of<QN>(s.vel)) * pstride, s.idx, g[i]);
  });
}

// ---------------------------------------------------------------- x-shifts without partial cache lines
// On an odd step (and in the push and adjoint kernels) population i moves by
// c_i. Addressed directly, the 18 populations with c_x != 0 are read and
// written one 4-byte element off the 256-byte segment of their wave, so every
// such access of a wave touches three cache lines, two of them partly; on
// rows longer than one wave the neighbouring wave completes those lines later
// and, on large lattices, after they have left the cache. Instead every lane
// accesses its own x (y and z shifted as before) and the values move by one
// lane inside the wave (a DPP rotation of the whole wave); the lane at the
// wave's edge takes its value from the neighbouring wave of the same row,
// through LDS. A block must hold whole rows (64 < n <= block size; x is the
// fastest index, so a row is n/64 consecutive waves). For n = 64 the row is
// one wave and the direct addresses already stay inside the wave's segment.

// lane l receives the value of lane l - 1 (lane 0: lane 63)
__device__ __forceinline__ uint32_t rot_from_prev(uint32_t v) {
  return uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x13C /* wave_ror:1 */, 0xF, 0xF, false));
}
// lane l receives the value of lane l + 1 (lane 63: lane 0)
__device__ __forceinline__ uint32_t rot_from_next(uint32_t v) {
  return uint32_t(__builtin_amdgcn_update_dpp(0, int(v), 0x134 /* wave_rol:1 */, 0xF, 0xF, false));
}
template <bool PREV, typename T>
__device__ __forceinline__ T rotate_lanes(T v) {
  if constexpr (sizeof(T) == 4) {
    const uint32_t u = __builtin_bit_cast(uint32_t, v);
    return __builtin_bit_cast(T, PREV ? rot_from_prev(u) : rot_from_next(u));
  } else {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = uint32_t(u), hi = uint32_t(u >> 32);
    const uint32_t rl = PREV ? rot_from_prev(lo) : rot_from_next(lo);
    const uint32_t rh = PREV ? rot_from_prev(hi) : rot_from_next(hi);
    return __builtin_bit_cast(T, (uint64_t(rh) << 32) | rl);
  }
}

// LDS for one exchange: per wave, the 9 values leaving through lane 63
// (towards +x) and the 9 leaving through lane 0 (towards -x)
template <typename T, int BLOCK>
using EdgeLds = T[BLOCK / 64][2][9];

// v[i] <- v[i] of node x - DIR * c_i,x of the same row (periodic), for every
// population i with c_i,x != 0. DIR = +1: values follow their velocity
// (streaming); DIR = -1: values are pulled from x + c_i (adjoint).
// Must be called by every thread of the block (it contains a barrier).
template <int QN, int DIR, int BLOCK, typename T>
__device__ __forceinline__ void row_shift(T (&v)[Q], EdgeLds<T, BLOCK>& edge, uint32_t n) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int wpr = int(n >> 6), rw = w & (wpr - 1), base = w - rw;
  const int prev = base + ((rw + wpr - 1) & (wpr - 1)), next = base + ((rw + 1) & (wpr - 1));
  for_vel<QN>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    constexpr int d = cx(i) * DIR;
    if constexpr (d == 1) {
      if (lane == 63) edge[w][0][i % 9] = v[i];
    } else if constexpr (d == -1) {
      if (lane == 0) edge[w][1][i % 9] = v[i];
    }
  });
  __syncthreads();
  for_vel<QN>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    constexpr int d = cx(i) * DIR;
    if constexpr (d == 1) {
      const T r = rotate_lanes<true>(v[i]);
      const T e = edge[prev][0][i % 9];
      v[i] = lane == 0 ? e : r;
    } else if constexpr (d == -1) {
      const T r = rotate_lanes<false>(v[i]);
      const T e = edge[next][1][i % 9];
      v[i] = lane == 63 ? e : r;
    }
  });
}

// index of x + s * (0, c_i,y, c_i,z): the node of the same x in the shifted row
template <int i, int s>
__host__ __device__ __forceinline__ uint32_t neighbour_yz(const Cell& c) {
  return c.oz[1 + s * cz(i)] + c.oy[1 + s * cy(i)] + c.ox[1];
}

__host__ __device__ __forceinline__ int remap_block(int b, int total, int xcd_remap) {
  // hardware dispatches workgroup b to XCD b % 8; give each XCD a contiguous run
  if (xcd_remap) {
    const int g8 = total & ~7;
    if (b < g8) b = (b & 7) * (g8 >> 3) + (b >> 3);
  }
  return b;
}

__host__ __device__ __forceinline__ int find_segment(const Seg* segs, int nseg, int b) {
  int lo = 0, hi = nseg - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (segs[mid].first_block <= b) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// The rows of a launch's segments of more than `chunk` blocks in chunks, by windows
// of `chunk` of the launch's blocks: the chunk that starts in window `window`
// ({0, 0} where none does). Segments that long hold a power of two of chunks,
// at least two, so at most one chunk starts in a window, and a segment that
// starts in a window holds the window's last block.
struct BlockChunk {
  int32_t first, count;  // block within the launch
};
__host__ __device__ __forceinline__ BlockChunk chunk_in_window(const Seg* segs, int nseg, int total_blocks, int chunk,
                                                               int window) {
  const int w = window * chunk, e = w + chunk < total_blocks ? w + chunk - 1 : total_blocks - 1;
  const Seg b = segs[find_segment(segs, nseg, e)];
  if (b.nblocks > chunk) {
    const int start = b.first_block + (e - b.first_block) / chunk * chunk;
    return start >= w ? BlockChunk{start, chunk} : BlockChunk{0, 0};
  }
  const Seg a = segs[find_segment(segs, nseg, w)];
  if (a.nblocks > chunk) {
    const int start = a.first_block + (w - a.first_block + chunk - 1) / chunk * chunk;
    if (start < a.first_block + a.nblocks) return {start, chunk};
  }
  return {0, 0};
}

// a value that is the same in every lane, in scalar registers
__device__ __forceinline__ uint32_t uniform32(uint32_t v) {
  return uint32_t(__builtin_amdgcn_readfirstlane(int(v)));
}
__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
  return (uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(v >> 32))))) << 32) |
         uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(v))));
}

// What a block of a step kernel works on.
struct BlockSite {
  int32_t sample;
  int32_t log2n;
  int32_t parity;
  uint32_t local_block;   // block within the sample
  uint32_t pstride;
  uint64_t offset;        // element offset of the sample's populations
};
__device__ __forceinline__ BlockSite block_site(const UniformSegs& u, int b) {
  const int s = b >> u.shift;
  return {u.sample0 + s, u.log2n, u.parity, uint32_t(b - (s << u.shift)), u.pstride, u.offset0 + uint64_t(s) * u.stride};
}
__device__ __forceinline__ BlockSite block_site(const Seg* segs, int nseg, const DevSample* samples, int b) {
  const Seg sg = segs[find_segment(segs, nseg, b)];
  const DevSample& sp = samples[sg.sample];
  return {sg.sample, sp.log2n, sg.parity, uint32_t(b - sg.first_block), sp.pstride, sp.offset};
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ double wave_min(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}

// Block reduction of the record quantities: 6 sums, 1 min, 1 max.
template <int BLOCK>
__device__ __forceinline__ void block_record(double (&v)[kRecord], double* out) {
  __shared__ double sh[BLOCK / 64][kRecord];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < 6; ++k) v[k] = wave_sum(v[k]);
  v[6] = wave_min(v[6]);
  v[7] = wave_max(v[7]);
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < kRecord; ++k) sh[wave][k] = v[k];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double r[kRecord];
#pragma unroll
    for (int k = 0; k < kRecord; ++k) r[k] = sh[0][k];
    for (int w = 1; w < BLOCK / 64; ++w) {
#pragma unroll
      for (int k = 0; k < 6; ++k) r[k] += sh[w][k];
      r[6] = fmin(r[6], sh[w][6]);
      r[7] = fmax(r[7], sh[w][7]);
    }
#pragma unroll
    for (int k = 0; k < kRecord; ++k) out[k] = r[k];
  }
}

}  // namespace
}  // namespace mclbm
