// The dyad of a dipole pair applied to moments in registers, for the kernels
// that re-evaluate it for every pair (fields at probes, matrix-free product,
// far-field double sum).  They are bound by the FP64 vector rate, so what counts
// is the number of instructions per pair: the dyad's three radial functions take
// about 60 (one reciprocal square root, one sine and cosine), and its products
// go through R (R . p) and R x p (28 and 24) instead of 3 x 3 matrices (54 and 36
// with 18 to form them).
//
// With n^2 = eps_env, P = p / n and N = n E the dyad is symmetric between the
// electric and magnetic parts,
//   N += a P + b R (R . P) - v R x m,   H += a m + b R (R . m) + v R x P,
//   a = e^{ikR} (k^2/R - 1/R^3 + ik/R^2),  b = e^{ikR} (-k^2/R + 3/R^3 - 3ik/R^2) / R^2,
//   v = e^{ikR} (k^2/R^2 + ik/R^3)
// (eps G^Ep = a I + b R R^T, n G^Hp = v [R]x).
#pragma once
#include "gdm_common.hpp"

namespace gdm {

// sin and cos of x + xl for 0 <= x <= 2^50 (larger ones are taken as 2^50), xl below
// an ulp of x, to about an ulp of 1: x - q pi in two parts of pi (Cody and Waite's
// reduction, with fused multiply-adds), then polynomials in (x - q pi)^2 on [0, (pi/2)^2], interpolated
// at Chebyshev nodes in 60 digits (absolute error below 2.3e-17).  q's parity
// comes out of the low bit of x / pi + 1.5 2^52.
__device__ inline void sincos_pos(double x, double xl, double& s, double& c) {
  x = fmin(x, 1125899906842624.0);
  const double t = fma(x, 0.3183098861837907, 6755399441055744.0);
  const double q = t - 6755399441055744.0;
  const double r = fma(-q, 3.141592653589793, x) + fma(-q, 1.2246467991473532e-16, xl);
  const double z = r * r;
  double u = 2.72157494212134e-15;
  u = fma(u, z, -7.643026557955253e-13);
  u = fma(u, z, 1.6058940878485947e-10);
  u = fma(u, z, -2.5052106890569507e-08);
  u = fma(u, z, 2.7557319211229606e-06);
  u = fma(u, z, -1.9841269841208676e-04);
  u = fma(u, z, 8.333333333333186e-03);
  u = fma(u, z, -0.16666666666666666);
  u = fma(r * z, u, r);
  double v = 4.627675984719231e-14;
  v = fma(v, z, -1.1464689885696053e-11);
  v = fma(v, z, 2.0876630867422246e-09);
  v = fma(v, z, -2.7557317767320517e-07);
  v = fma(v, z, 2.4801587292446213e-05);
  v = fma(v, z, -1.3888888888860709e-03);
  v = fma(v, z, 4.166666666666634e-02);
  v = fma(v, z, -0.5);
  v = fma(v, z, 1.0);
  const int flip = __double2loint(t) << 31;
  s = __hiloint2double(__double2hiint(u) ^ flip, __double2loint(u));
  c = __hiloint2double(__double2hiint(v) ^ flip, __double2loint(v));
}

struct Dyad {
  double2 a, b, v;
};

// The radial functions at |R|^2 = R2 > 0 (v only if WANT_V).
template <bool WANT_V> __device__ inline Dyad dyad_at(double R2, double k) {
  // 1/R: the hardware's approximation (about 2^-23) with one third-order step.
  // The phase k R goes on in two parts: rounded to one it would be off by half an
  // ulp of itself, the largest error of a distant pair (E of 4784 dipoles against
  // 80-bit sums: 2.1e-15; by a kernel that rounded it once 4.7e-15).
  double y = __builtin_amdgcn_rsq(R2);
  const double e = fma(-R2 * y, y, 1.0);
  y = fma(y * e, fma(e, 0.375, 0.5), y);
  const double R = R2 * y, Rl = fma(-R, R, R2) * (0.5 * y);
  const double x = k * R;
  double s, c;
  sincos_pos(x, fma(k, Rl, fma(k, R, -x)), s, c);
  const double y2 = y * y, k2 = k * k;
  const double ai = k * y2, ar = y * (k2 - y2);
  const double y3 = y2 * y;
  const double br = y3 * fma(3.0, y2, -k2), bi = ai * (-3.0 * y2);
  Dyad d;
  d.a = make_double2(fma(c, ar, -s * ai), fma(c, ai, s * ar));
  d.b = make_double2(fma(c, br, -s * bi), fma(c, bi, s * br));
  if (WANT_V) {
    const double vr = k2 * y2, vi = k * y3;
    d.v = make_double2(fma(c, vr, -s * vi), fma(c, vi, s * vr));
  }
  return d;
}

__device__ inline void zfma(double2& a, const double2& b, const double2& c) {
  a.x = fma(-b.y, c.y, fma(b.x, c.x, a.x));
  a.y = fma(b.y, c.x, fma(b.x, c.y, a.y));
}

// F += a p + b R (R . p)
__device__ inline void dyad_electric(double2 (&F)[3], const Dyad& d, const double (&R)[3], const double2& px,
                                     const double2& py, const double2& pz) {
  const double tx = fma(R[2], pz.x, fma(R[1], py.x, R[0] * px.x));
  const double ty = fma(R[2], pz.y, fma(R[1], py.y, R[0] * px.y));
  const double2 t = make_double2(fma(d.b.x, tx, -d.b.y * ty), fma(d.b.x, ty, d.b.y * tx));
  const double2 p[3] = {px, py, pz};
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    F[i].x = fma(R[i], t.x, F[i].x);
    F[i].y = fma(R[i], t.y, F[i].y);
    zfma(F[i], d.a, p[i]);
  }
}

// F += (+1, -1) v R x p
template <int SIGN>
__device__ inline void dyad_magnetic(double2 (&F)[3], const Dyad& d, const double (&R)[3], const double2& px,
                                     const double2& py, const double2& pz) {
  const double2 p[3] = {px, py, pz};
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const int j = (i + 1) % 3, k = (i + 2) % 3;
    // SIGN (R x p)_i
    const double cx = SIGN > 0 ? fma(R[j], p[k].x, -R[k] * p[j].x) : fma(R[k], p[j].x, -R[j] * p[k].x);
    const double cy = SIGN > 0 ? fma(R[j], p[k].y, -R[k] * p[j].y) : fma(R[k], p[j].y, -R[j] * p[k].y);
    zfma(F[i], d.v, make_double2(cx, cy));
  }
}

}  // namespace gdm
