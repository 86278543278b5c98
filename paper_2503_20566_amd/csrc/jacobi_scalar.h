// The parts of the one-sided Jacobi (row_sweep.h) that are plain functions of numbers: the LDS layout of the
// column scales and the arithmetic of a rotation.  Nothing here names a thread or a memory space, so that a host
// compiler takes them too.
#pragma once

namespace gipeps {

// every multiply-add is written as fma where it is one (row_sweep.h)
#pragma clang fp contract(off)

// Where the column scales (d, 1/d) lie in LDS, in entries of two doubles, for ng column groups.  Three ranges
// that share no entry:
//   lower(k)  the scales of group k's first column, which group k - 1 reads between the two barriers of a
//             boundary round;
//   upper(k)  those of the column that group k hands up, which group k + 1 reads after the second barrier;
//   end(p)    at the end of a sweep, the scales of slots 2 p and 2 p + 1, for the J rows.
// No barrier lies between a sweep's last read of upper and its first write of end, and reader and writer are
// in different waves from 33 columns on: with end over lower and upper, a group of four columns, which writes
// two entries of end, could overwrite an entry of upper that another wave had still to read.
struct JacobiScales {
  int ng;
  constexpr int lower(int k) const { return k; }
  constexpr int upper(int k) const { return ng + k; }
  constexpr int end(int p) const { return 2 * ng + p; }
  // entries for up to maxn columns in groups of nc
  static constexpr int room(int maxn, int nc) { return 2 * (maxn / nc) + maxn / 2; }
};

// ---------------------------------------------------------------------------------------------
// Rotation arithmetic of the Jacobi step.  The Jacobi scales its matrix by a power of two so that
// ||A||_F^2 is of order one, which keeps every argument below a normal number far from the
// exponent limits; the square root and reciprocal therefore use the hardware estimates refined by
// Newton steps, without the rescaling and special-value handling of the library routines.
// ---------------------------------------------------------------------------------------------
// t = tan(theta) of the smaller rotation angle annihilating a_i.a_j, from dd = |a_j|^2 - |a_i|^2
// and g2 = 2 a_i.a_j (g2 != 0): t = sign(dd) g2 / (|dd| + sqrt(dd^2 + g2^2)), within 4 x 2^-53.  The hardware
// estimates are good to 2^-24 (measured): the square root takes a Goldschmidt step and a correction by its
// residual, the quotient a Newton step of the reciprocal and a correction.  (With one step each and no
// corrections t was off by up to 50 ulp, 12 rms, now 3.1 and 0.6.  They cost: energy at 6 x 6, chi 6, 33 samples,
// 778 -> 788 us; gradient at 16 x 16, chi 16, 1024 samples, 43.35 -> 43.58 ms.)
__device__ __forceinline__ double rotation_tangent(double dd, double g2) {
  const double x = fma(dd, dd, g2 * g2);
  const double y0 = __builtin_amdgcn_rsq(x);
  const double h = 0.5 * y0;
  double g = x * y0;
  g = fma(g, fma(-g, h, 0.5), g);
  const double den = fabs(dd) + fma(fma(-g, g, x), h, g);  // g corrected: sqrt(x)
  double y = __builtin_amdgcn_rcp(den);
  y = fma(y, fma(-den, y, 1.0), y);
  const double s = dd < 0.0 ? -g2 : g2;
  const double q = s * y;
  return fma(fma(-den, q, s), y, q);  // q corrected by its residual
}

// 1 / sqrt(a) for a in [1, 2], rounded (within 2^-54 but for terms of the order of 2^-77): the estimate and one
// third-order step, y (1 + e/2 + 3 e^2/8) with e = 1 - a y^2, a y with its low part.  Without the low part the
// error is not larger than 2^-53, but it has a sign: just above 1 the estimate is 1 - 2^-53 and a y rounds the same
// way each time, so that every small rotation made its columns longer by 2^-53 (mean error 0.67 x 2^-53 near 1,
// now 0.00; 0.37 with two Newton steps).  Over the rotations of 128 columns graded over eight decades J was up to
// 8e-14 from orthogonal, now 1.3e-14.  Same time within the runs' spread.
__device__ __forceinline__ double rsqrt_1to2(double a) {
  const double y = __builtin_amdgcn_rsq(a);
  const double p = a * y;
  const double e = fma(-fma(a, y, -p), y, fma(-p, y, 1.0));
  return fma(y * e, fma(0.375, e, 0.5), y);
}

// A column's squared norm (carried, not recomputed), its scale and the scale's inverse
struct Col {
  double n, d, id;
};
// The rotation of the pair (u, v) from u^ . v^ (gs): the factors of the scaled update, u^' = u^ - alpha v^
// and v^' = v^ + beta u^ (0 when the pair is left alone); norms and scales are advanced.
struct PairRot {
  double alpha, beta;
  bool on;
};
__device__ __forceinline__ PairRot pair_rotation(double gs, Col& u, Col& v, double zero2, double tol2, bool& big_any) {
  constexpr double kQuadratic2 = 1e-12;  // (1e-6)^2
  const double g = gs * (u.d * v.d);
  const double gg = g * g, ab = u.n * v.n;
  const bool pos = fmin(u.n, v.n) > zero2;
  big_any |= pos && gg > kQuadratic2 * ab;
  PairRot r{0.0, 0.0, pos && gg > tol2 * ab};
  if (r.on) {
    const double t = rotation_tangent(v.n - u.n, g + g);
    const double a = fma(t, t, 1.0);
    const double c = rsqrt_1to2(a), ic = a * c;
    r.alpha = t * (v.d * u.id);
    r.beta = t * (u.d * v.id);
    u.n = fma(-t, g, u.n);
    v.n = fma(t, g, v.n);
    u.d *= c;
    v.d *= c;
    u.id *= ic;
    v.id *= ic;
  }
  return r;
}

// Two pairs at once, without a branch between them, so that their chains (a hundred dependent instructions
// each) interleave; a pair left alone gets the factors 0 and keeps its norms and scales.
__device__ __forceinline__ void pair_rotations(double gs0, double gs1, Col& u0, Col& v0, Col& u1, Col& v1, double zero2,
                                               double tol2, bool& big_any, PairRot& r0, PairRot& r1) {
  constexpr double kQuadratic2 = 1e-12;
  const double g0 = gs0 * (u0.d * v0.d), g1 = gs1 * (u1.d * v1.d);
  const double gg0 = g0 * g0, ab0 = u0.n * v0.n, gg1 = g1 * g1, ab1 = u1.n * v1.n;
  const bool pos0 = fmin(u0.n, v0.n) > zero2, pos1 = fmin(u1.n, v1.n) > zero2;
  big_any |= (pos0 && gg0 > kQuadratic2 * ab0) || (pos1 && gg1 > kQuadratic2 * ab1);
  r0 = PairRot{0.0, 0.0, pos0 && gg0 > tol2 * ab0};
  r1 = PairRot{0.0, 0.0, pos1 && gg1 > tol2 * ab1};
  if (r0.on || r1.on) {
    double t0 = rotation_tangent(v0.n - u0.n, g0 + g0), t1 = rotation_tangent(v1.n - u1.n, g1 + g1);
    t0 = r0.on ? t0 : 0.0;
    t1 = r1.on ? t1 : 0.0;
    const double a0 = fma(t0, t0, 1.0), a1 = fma(t1, t1, 1.0);
    double c0 = rsqrt_1to2(a0), c1 = rsqrt_1to2(a1);
    c0 = r0.on ? c0 : 1.0;
    c1 = r1.on ? c1 : 1.0;
    const double ic0 = a0 * c0, ic1 = a1 * c1;
    r0.alpha = t0 * (v0.d * u0.id);
    r0.beta = t0 * (u0.d * v0.id);
    r1.alpha = t1 * (v1.d * u1.id);
    r1.beta = t1 * (u1.d * v1.id);
    u0.n = fma(-t0, g0, u0.n);
    v0.n = fma(t0, g0, v0.n);
    u1.n = fma(-t1, g1, u1.n);
    v1.n = fma(t1, g1, v1.n);
    u0.d *= c0;
    v0.d *= c0;
    u1.d *= c1;
    v1.d *= c1;
    u0.id *= ic0;
    v0.id *= ic0;
    u1.id *= ic1;
    v1.id *= ic1;
  }
}

}  // namespace gipeps
