// sblm_math.h -- the arithmetic of one magnification and one fit update
// (Rajpaul 2012, Sec. 2.2 and Sec. 4.4): source position, lens polynomial,
// Ehrlich-Aberth sweep, image evaluation and refinement on the lens
// equation, least-squares row update.
//
// Written once for any number type R and shared by two builds: the fitness
// kernel (device code, R = double or float) and the FLOP counting build
// (host code, R = a number type that counts its operations), so that the
// operation counts used for the roofline come from this very code.  Every R
// supplies, found by overload resolution: fma(a, b, c), rcp_hw(x) and rsq_hw(x)
// (the hardware estimates of 1/x and 1/sqrt(x)), vmin / vmax (minimum / maximum), fabs and
// isfinite; is_single<R> says whether R stands for FP32 (its reciprocal
// steps take no refinement).
#pragma once

#ifdef __HIP__
#define SBLM_FN __host__ __device__ __forceinline__
#else
#define SBLM_FN inline
#endif

namespace sblm {

template <typename R>
struct is_single {
  static constexpr bool value = false;
};
template <>
struct is_single<float> {
  static constexpr bool value = true;
};

// ---------------------------------------------------------------- reciprocals

// Raw hardware reciprocal (relative error < 5e-8 in FP64): used only for the
// pairwise terms of the Aberth correction, whose error scales the size of a
// correction that is itself second order.
template <typename R>
SBLM_FN R rcp_raw(R x) {
  return rcp_hw(x);
}
// Approximate reciprocal for iteration steps (the fixed point of the
// iteration does not depend on its accuracy): FP64 one Newton step on the
// estimate, FP32 the estimate.
template <typename R>
SBLM_FN R rcp_fast(R x) {
  if constexpr (is_single<R>::value) {
    return rcp_hw(x);
  } else {
    const R r = rcp_hw(x);
    return fma(r, fma(-x, r, R(1.0)), r);
  }
}
// Reciprocal to about 1 ulp (two Newton steps), for det J, image positions
// and the fit.
template <typename R>
SBLM_FN R rcp_acc(R x) {
  R r = rcp_hw(x);
  r = fma(r, fma(-x, r, R(1.0)), r);
  return fma(r, fma(-x, r, R(1.0)), r);
}

// ---------------------------------------------------------------- complex

template <typename T>
struct cx {
  T re, im;
};

template <typename T>
SBLM_FN cx<T> c_sub(cx<T> a, cx<T> b) {
  return {a.re - b.re, a.im - b.im};
}
// a*b + c
template <typename T>
SBLM_FN cx<T> c_fma(cx<T> a, cx<T> b, cx<T> c) {
  return {fma(a.re, b.re, fma(-a.im, b.im, c.re)), fma(a.re, b.im, fma(a.im, b.re, c.im))};
}
template <typename T>
SBLM_FN cx<T> c_mul(cx<T> a, cx<T> b) {
  return {fma(a.re, b.re, -a.im * b.im), fma(a.re, b.im, a.im * b.re)};
}
template <typename T>
SBLM_FN T c_norm(cx<T> a) {
  return fma(a.re, a.re, a.im * a.im);
}

// ---------------------------------------------------------------- polynomial

// Source position of Eq. (sourcePos) at dimensionless time tau = (t - t0)/tE
// (itE = 1/tE), trajectory angle alpha (sa = sin, ca = cos), impact u0.
template <typename R>
SBLM_FN cx<R> source_position(R t, R t0, R itE, R sa, R ca, R u0) {
  const R tau = (t - t0) * itE;
  return {fma(tau, sa, u0 * ca), fma(-tau, ca, u0 * sa)};
}

// Coefficients c[0..5] of the lens polynomial for source zeta, separation d,
// mass ratio q.  From Eq. (lensing): conj(z) = N(z)/D(z) with
// N = w z^2 + (1+q-dw) z - d, D = z^2 - d z, w = conj(zeta); substituting
// back and clearing denominators gives (zeta - z) N M + M D + q N D = 0 with
// M = N - d D = (w-d) z^2 + (1+q+d^2-dw) z - d.  Expanded here by hand.
template <typename R>
SBLM_FN void lens_coeffs(cx<R> zeta, R d, R q, cx<R> c[6]) {
  const cx<R> w = {zeta.re, -zeta.im};
  const R opq = R(1.0) + q;
  const cx<R> n2 = w;
  const cx<R> n1 = {fma(-d, w.re, opq), -d * w.im};
  const cx<R> m2 = {w.re - d, w.im};
  const cx<R> m1 = {fma(-d, w.re, fma(d, d, opq)), -d * w.im};
  const R dd = d * d;
  // products of N and M, by power of z (n0 = m0 = -d)
  const cx<R> nm4 = c_mul(n2, m2);
  const cx<R> nm3 = c_fma(n2, m1, c_mul(n1, m2));
  const cx<R> s2 = {n2.re + m2.re, n2.im + m2.im};
  const cx<R> nm2 = c_fma(n1, m1, cx<R>{-d * s2.re, -d * s2.im});
  const cx<R> nm1 = {-d * (n1.re + m1.re), -d * (n1.im + m1.im)};
  // (zeta - z) N M + M D + q N D
  c[5] = {-nm4.re, -nm4.im};
  // z^4: zeta nm4 - nm3 + m2 + q n2
  c[4] = c_fma(zeta, nm4,
               cx<R>{m2.re + fma(q, n2.re, -nm3.re), m2.im + fma(q, n2.im, -nm3.im)});
  // z^3: zeta nm3 - nm2 + (m1 - d m2) + q (n1 - d n2)
  c[3] = c_fma(zeta, nm3,
               cx<R>{fma(-d, m2.re, m1.re) + fma(q, fma(-d, n2.re, n1.re), -nm2.re),
                     fma(-d, m2.im, m1.im) + fma(q, fma(-d, n2.im, n1.im), -nm2.im)});
  // z^2: zeta nm2 - nm1 + (m0 - d m1) + q (n0 - d n1)
  c[2] = c_fma(zeta, nm2,
               cx<R>{fma(-d, m1.re, -d) + fma(q, fma(-d, n1.re, -d), -nm1.re),
                     fma(-d, m1.im, R(0.0)) + fma(q, -d * n1.im, -nm1.im)});
  // z^1: zeta nm1 - nm0 - d m0 - q d n0 = zeta nm1 + q d^2
  c[1] = c_fma(zeta, nm1, cx<R>{q * dd, R(0.0)});
  // z^0: zeta nm0 = zeta d^2
  c[0] = {zeta.re * dd, zeta.im * dd};
}

// A negligible leading coefficient (the source on a lens): the polynomial is
// solved as one of degree 4 and c[5] is set to zero.
template <typename R>
SBLM_FN bool drop_to_degree4(cx<R> c[6]) {
  R cmax = R(0.0);
#pragma unroll
  for (int j = 0; j < 6; ++j) cmax = vmax(cmax, c_norm(c[j]));
  const bool deg4 = c_norm(c[5]) <= R(1e-24) * cmax;
  if (deg4) c[5] = {R(0.0), R(0.0)};
  return deg4;
}

// A source very close to a lens (within ~1e-3 theta_E of either) gives a
// small leading coefficient: one root -- always spurious -- lies far out, at
// about -c4/c5, the others near the lenses.  |c4| > 1e3 |c5| marks it.
template <typename R>
SBLM_FN bool far_root(const cx<R> c[6]) {
  return c_norm(c[4]) > R(1e6) * c_norm(c[5]);
}

// p(z) and p'(z) by Horner's rule.
template <typename T>
SBLM_FN void horner(const cx<T> c[6], cx<T> z, cx<T>& p, cx<T>& dp) {
  dp = c[5];
  p = c_fma(c[5], z, c[4]);
#pragma unroll
  for (int j = 3; j >= 0; --j) {
    dp = c_fma(dp, z, p);
    p = c_fma(p, z, c[j]);
  }
}

// One Ehrlich-Aberth sweep (Jacobi form) over the five roots:
//   S_i = sum_{j != i} 1/(z_i - z_j),
//   z_i <- z_i - p(z_i) / (p'(z_i) - p(z_i) S_i),
// (the usual w/(1 - w S) with w = p/p', written with one complex division).
// The iteration converges cubically: after a step of length e the error
// left in z_i is about e^3 / s_i^2, s_i the distance to the nearest other
// root.  Returns 1 when, for every root, e^3 / (s_i^2 max(1,|z_i|)) <= tau or
// e <= 1e-13 max(1,|z_i|) (a step at the rounding level, which also ends the
// slow approach of a double root).  With EM, *emax receives
// max_i e_i^2 / max(1,|z_i|^2) (a termination heuristic: the raw reciprocal,
// no division); without, emax is not touched.
template <bool EM = true, typename T>
SBLM_FN bool aberth_sweep(const cx<T> c[6], cx<T> z[5], bool deg4, T tau, T* emax) {
  // pairwise terms from the current roots first, so that each root's p, p'
  // is used as soon as it is computed (fewer live registers)
  cx<T> S[5];
  T dmin[5];  // (distance to the nearest other root)^2
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    S[i] = {T(0.0), T(0.0)};
    dmin[i] = T(INFINITY);
  }
#pragma unroll
  for (int i = 0; i < 5; ++i)
#pragma unroll
    for (int j = i + 1; j < 5; ++j) {
      const cx<T> dz = c_sub(z[i], z[j]);
      const T n = c_norm(dz);
      const T r = rcp_raw(n);
      const T ire = dz.re * r, iim = -dz.im * r;  // 1/(z_i - z_j)
      S[i].re += ire;
      S[i].im += iim;
      S[j].re -= ire;
      S[j].im -= iim;
      dmin[i] = vmin(n, dmin[i]);
      dmin[j] = vmin(n, dmin[j]);
    }
  bool conv = true;
  T em = T(0.0);
  const T tau2 = tau * tau;
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    cx<T> p, dp;
    horner(c, z[i], p, dp);
    // den = p' - p S ; dz = p / den
    const cx<T> pS = c_mul(p, S[i]);
    const cx<T> den = c_sub(dp, pS);
    const T r = rcp_fast(c_norm(den));
    cx<T> dz = {fma(p.re, den.re, p.im * den.im) * r, fma(p.im, den.re, -p.re * den.im) * r};
    if (i == 4 && deg4) dz = {T(0.0), T(0.0)};
    z[i] = c_sub(z[i], dz);
    const T zn = c_norm(z[i]);
    const T sc = vmax(zn, T(1.0));
    const T e2 = c_norm(dz);
    // (e^2)^3 <= tau^2 |z|^2 (s^2)^2, or e^2 <= 1e-26 |z|^2
    const bool ok = (e2 * e2 * e2 <= tau2 * sc * (dmin[i] * dmin[i])) || (e2 <= T(1e-26) * sc);
    conv = conv && (ok || (i == 4 && deg4));
    if constexpr (EM) em = vmax(e2 * rcp_raw(sc), em);
  }
  if constexpr (EM) *emax = em;
  return conv;
}

// Squared distance from each root to its nearest other root.
template <typename T>
SBLM_FN void nearest2(const cx<T> z[5], T d2[5]) {
#pragma unroll
  for (int i = 0; i < 5; ++i) d2[i] = T(INFINITY);
#pragma unroll
  for (int i = 0; i < 5; ++i)
#pragma unroll
    for (int j = i + 1; j < 5; ++j) {
      const T n = c_norm(c_sub(z[i], z[j]));
      d2[i] = vmin(n, d2[i]);
      d2[j] = vmin(n, d2[j]);
    }
}

// One Newton step on every root, z_i <- z_i - p(z_i)/p'(z_i) (the polish of
// roots found in lower precision).  Newton's method converges
// quadratically: after a step of length e the error left is about e^2/s_i
// (s_i the distance to the nearest other root, from d2).  Returns 1 when,
// for every root, e^2/s_i <= tau max(1,|z_i|), i.e. e^4 <= tau^2 |z_i|^2
// s_i^2, or e <= 1e-13 max(1,|z_i|) (a step at the rounding level).
template <typename T>
SBLM_FN bool newton_pass(const cx<T> c[6], cx<T> z[5], const T d2[5], T tau) {
  bool conv = true;
  const T tau2 = tau * tau;
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    cx<T> p, dp;
    horner(c, z[i], p, dp);
    const T r = rcp_fast(c_norm(dp));
    const cx<T> dz = {fma(p.re, dp.re, p.im * dp.im) * r, fma(p.im, dp.re, -p.re * dp.im) * r};
    z[i] = c_sub(z[i], dz);
    const T sc = vmax(c_norm(z[i]), T(1.0));
    const T e2 = c_norm(dz);
    conv = conv && ((e2 * e2 <= tau2 * sc * d2[i]) || (e2 <= T(1e-26) * sc));
  }
  return conv;
}

// ---------------------------------------------------------------- images

#define SBLM_IMAGE_TOL2 1e-12 /* residual threshold 1e-6, squared */
#define SBLM_POLISH_DETJ 0.01 /* images with |det J| below this are refined */
#define SBLM_POLISH_EST2 1e-24 /* ... and those whose residual could move A by \
                                  more than 1e-12 relative (squared) */

// Lens-equation quantities at a trial image z: the residual
// r = zeta - z + 1/conj(z) - q/(d - conj(z)) of Eq. (lensing) and
// g = dzeta/dconj(z) = 1/conj(z)^2 + q/(d - conj(z))^2; returns |r|^2.
// *iz2, *ie2 receive |1/z|^2 and |1/(d - z)|^2.
template <typename R>
SBLM_FN R image_eval(cx<R> z, cx<R> zeta, R d, R q, cx<R>& res, cx<R>& g, R* iz2, R* ie2) {
  const R x = z.re, y = z.im;
  // a = 1/conj(z) = z / |z|^2 ; b = 1/(d - conj(z))
  // one reciprocal for both: 1/|z|^2 = |d-z|^2 / P, 1/|d-z|^2 = |z|^2 / P with
  // P = |z|^2 |d-z|^2 (within range: |z| stays far from the FP64 limits)
  const R n2 = fma(x, x, y * y);
  const R ex = d - x;
  const R e2 = fma(ex, ex, y * y);
  const R ip = rcp_acc(n2 * e2);
  const R iz = e2 * ip;
  const cx<R> a = {x * iz, y * iz};
  const R ie = n2 * ip;
  const cx<R> b = {ex * ie, -y * ie};
  res = {fma(-q, b.re, (zeta.re - x) + a.re), fma(-q, b.im, (zeta.im - y) + a.im)};
  const cx<R> b2 = c_mul(b, b);
  g = c_fma(a, a, cx<R>{q * b2.re, q * b2.im});
  *iz2 = iz;
  *ie2 = ie;
  return c_norm(res);
}

// The image test of one root: its squared residual *r2 on the lens equation,
// |det J| (*adet), and whether the image needs refining: when it lies very
// close to a critical curve (|det J| < 0.01) or when its residual r could
// move A by more than 1e-12 relative -- the image moves by about
// (1 + |g|) |r| / |det J|, det J by 2 |g| |h| times that
// (h = dg/dconj(z), |h| <= 2|1/z|^3 + 2q|1/(d-z)|^3) and A_i by A_i^2 times
// that, with A >= 1.
template <typename R>
SBLM_FN bool image_score(cx<R> z, cx<R> zeta, R d, R q, R* r2, R* adet) {
  cx<R> res, g;
  R iz2, ie2;
  *r2 = image_eval(z, zeta, d, q, res, g, &iz2, &ie2);
  const R gn = c_norm(g);
  *adet = fabs(R(1.0) - gn);
  // (dA/A)^2 <= 64 |g|^2 (1 + |g|^2) (|1/z|^6 + q^2 |1/(d-z)|^6) |r|^2 / |det J|^6;
  // refine when that exceeds SBLM_POLISH_EST2 (compared without dividing)
  const R a3 = *adet * *adet * *adet;
  const R num = R(64.0) * gn * (R(1.0) + gn) * fma(q * q * ie2, ie2 * ie2, iz2 * iz2 * iz2) * *r2;
  return !(num <= R(SBLM_POLISH_EST2) * (a3 * a3)) || *adet < R(SBLM_POLISH_DETJ);
}

// One image refined by up to two Newton steps on the lens equation itself,
// dz = (r - g conj(r))/(1 - |g|^2), each kept only if it lowers the
// residual; returns its 1/|det J|.  Near a critical curve (near-coincident
// roots next to a caustic) or in the root cluster around the secondary lens
// at small q the quintic's roots lose accuracy, while the lens equation does
// not.
template <typename R>
SBLM_FN R refine_image(cx<R> zi, cx<R> zeta, R d, R q) {
  cx<R> res, g;
  R iz2, ie2;
  R rn = image_eval(zi, zeta, d, q, res, g, &iz2, &ie2);
  for (int step = 0; step < 2; ++step) {
    const R det = R(1.0) - c_norm(g);
    const R idet = rcp_acc(det);
    // dz = (r - g conj(r)) / det
    const cx<R> gr = c_mul(g, cx<R>{res.re, -res.im});
    const cx<R> dz = {(res.re - gr.re) * idet, (res.im - gr.im) * idet};
    const cx<R> zn = {zi.re + dz.re, zi.im + dz.im};
    cx<R> resn, gn2;
    const R rnn = image_eval(zn, zeta, d, q, resn, gn2, &iz2, &ie2);
    if (!(rnn < rn)) break;
    zi = zn;
    res = resn;
    g = gn2;
    rn = rnn;
    // Newton converges quadratically: after a step of 1e-10 |z| the next
    // one would be at the rounding level
    if (c_norm(dz) <= R(1e-20) * c_norm(zi)) break;
  }
  return rcp_acc(fabs(R(1.0) - c_norm(g)));
}

// ---------------------------------------------------------------- tracking

// At most epochs of a chain the images move a little and none appears or
// vanishes.  Then three images followed on the lens equation itself (Newton
// from their extrapolation) give the other two roots of the lens polynomial
// in closed form, from the sum and the product of all five, and with them
// the image count: no simultaneous iteration.  Any three distinct solutions of
// the lens equation will do -- they are roots of the polynomial -- so a step
// only has to show that it has arrived at one (image_close, whose two bounds
// together prove it); where it cannot (next to a caustic, after a long gap, a
// source on a lens) the five roots are solved for.

// Square root to about 1 ulp from the hardware estimate of 1/sqrt(x) (x > 0).
template <typename R>
SBLM_FN R sqrt_acc(R x) {
  const R y = rsq_hw(x);
  R g = x * y, h = R(0.5) * y;
  const R e = fma(-h, g, R(0.5));
  g = fma(g, e, g);
  h = fma(h, e, h);
  return fma(fma(-g, g, x), h, g);
}

#define SBLM_TRACK_EST 1e-12 /* relative error of an image's A after its last step */
#define SBLM_TRACK_STEP 1e-2 /* that step against the distance to a lens at most */
#define SBLM_TRACK_SPURIOUS2 1e-8 /* |residual|^2 above which a root is no image */
#define SBLM_TRACK_IMAGE2 1e-16   /* ... and below which it is one */
#define SBLM_TRACK_APART2 1e-10   /* |z_i - z_j|^2 of two images at least */

// The lens equation at a trial image z, as image_eval: residual r, g =
// a^2 + q b^2 with a = 1/conj(z), b = 1/(d - conj(z)).
template <typename R>
struct LensAt {
  cx<R> a, b, a2, qb2, r, g;
  R iz, ie;
};
template <bool ACC, typename R>
SBLM_FN LensAt<R> lens_at(cx<R> z, cx<R> zeta, R d, R q) {
  LensAt<R> e;
  const R x = z.re, y = z.im;
  const R n2 = fma(x, x, y * y);
  const R ex = d - x;
  const R e2 = fma(ex, ex, y * y);
  const R ip = ACC ? rcp_acc(n2 * e2) : rcp_fast(n2 * e2);
  e.iz = e2 * ip;
  e.ie = n2 * ip;
  e.a = {x * e.iz, y * e.iz};
  e.b = {ex * e.ie, -y * e.ie};
  e.r = {fma(-q, e.b.re, (zeta.re - x) + e.a.re), fma(-q, e.b.im, (zeta.im - y) + e.a.im)};
  e.a2 = c_mul(e.a, e.a);
  const cx<R> b2 = c_mul(e.b, e.b);
  e.qb2 = {q * b2.re, q * b2.im};
  e.g = {e.a2.re + e.qb2.re, e.a2.im + e.qb2.im};
  return e;
}

// |residual|^2 of the lens equation at z.
template <typename R>
SBLM_FN R lens_residual2(cx<R> z, cx<R> zeta, R d, R q) {
  const R x = z.re, y = z.im;
  const R n2 = fma(x, x, y * y);
  const R ex = d - x;
  const R e2 = fma(ex, ex, y * y);
  const R ip = rcp_fast(n2 * e2);
  const R iz = e2 * ip, qe = q * (n2 * ip);
  return c_norm(cx<R>{fma(x, iz, fma(-ex, qe, zeta.re - x)), fma(y, iz, fma(y, qe, zeta.im - y))});
}

// One Newton step on the lens equation, z += (r - g conj(r))/(1 - |g|^2).
template <typename R>
SBLM_FN void image_newton(cx<R>& z, cx<R> zeta, R d, R q) {
  const LensAt<R> e = lens_at<false>(z, zeta, d, q);
  const R id = rcp_raw(R(1.0) - c_norm(e.g));
  const cx<R> gr = c_mul(e.g, cx<R>{e.r.re, -e.r.im});
  z = {fma(e.r.re - gr.re, id, z.re), fma(e.r.im - gr.im, id, z.im)};
}

// A Newton step that is meant to be the last: *g is g after it to first order
// in dz, g + h conj(dz) with h = dg/dconj(z) = 2 q b^3 - 2 a^3, *inv the
// reciprocal of det J = 1 - |g|^2.  Returns whether z is an image and A_i =
// |1/det J| final:
//   - the step is at most SBLM_TRACK_STEP of the distance to either lens, so
//     that over all of it g's derivatives are those at its start to a few
//     percent.  Without this the next bound says nothing: a step taken at
//     |det J| = 0 throws z far out, where g = 0 and the step after it, z -> zeta,
//     passes it with no image there;
//   - what is neglected (|dz|^2 dg''/2 in g, and the position's remaining error
//     K |dz|^2, K = |h| (1 + |g|)/(2 |det|)) moves A_i by at most SBLM_TRACK_EST
//     relative.  K |dz| is then below 1e-6, so (Newton-Kantorovich) there is one
//     solution of the lens equation within two steps of the start, and z is
//     K |dz|^2 from it.
// (|g| <= (1 + |g|^2)/2 keeps square roots out of the bound; false for NaN.)
template <typename R>
SBLM_FN bool image_close(cx<R>& z, cx<R> zeta, R d, R q, cx<R>* g, R* inv) {
  const LensAt<R> e = lens_at<true>(z, zeta, d, q);
  const R gn = c_norm(e.g), det = R(1.0) - gn;
  const R id = rcp_fast(det);
  const cx<R> gr = c_mul(e.g, cx<R>{e.r.re, -e.r.im});
  const cx<R> dz = {(e.r.re - gr.re) * id, (e.r.im - gr.im) * id};
  // h/2 and g after the step
  const cx<R> a3 = c_mul(e.a2, e.a);
  const cx<R> hh = c_fma(e.qb2, e.b, cx<R>{-a3.re, -a3.im});
  const cx<R> dh = c_mul(hh, cx<R>{dz.re, -dz.im});
  *g = {fma(R(2.0), dh.re, e.g.re), fma(R(2.0), dh.im, e.g.im)};
  *inv = rcp_acc(R(1.0) - c_norm(*g));
  z = {z.re + dz.re, z.im + dz.im};
  const R dn = c_norm(dz), hn = c_norm(hh);
  const bool small = (R(1.0) + gn) * dn *
                         fma(R(3.0) * fma(e.iz, e.iz, q * e.ie * e.ie), fabs(det),
                             hn * (R(3.0) + gn)) <=
                     R(SBLM_TRACK_EST) * (det * det);
  return dn * (e.iz + e.ie) <= R(SBLM_TRACK_STEP * SBLM_TRACK_STEP) && small;
}

// The other two roots (z3, z4) of the lens polynomial from three of them, by
// the sum -c4/c5 and the product -c0/c5 of all five.  False where that loses
// accuracy: a root far out (|c4| > 1e3 |c5|), or the two closer than about
// 1e-4 of their mean.
template <typename R>
SBLM_FN bool other_roots(cx<R> zeta, R d, R q, const cx<R> z[3], cx<R>& z3, cx<R>& z4) {
  // c5 = -n2 m2, c4 = zeta n2 m2 - (n2 m1 + n1 m2) + m2 + q n2, c0 = zeta d^2
  // (lens_coeffs)
  const cx<R> w = {zeta.re, -zeta.im};
  const R opq = R(1.0) + q;
  const cx<R> n1 = {fma(-d, w.re, opq), -d * w.im};
  const cx<R> m2 = {w.re - d, w.im};
  const cx<R> m1 = {fma(d, d, n1.re), n1.im};
  const cx<R> c5 = c_mul(w, m2);  // -c5
  const cx<R> nm3 = c_fma(w, m1, c_mul(n1, m2));
  const cx<R> c4 = c_fma(zeta, c5, cx<R>{m2.re + fma(q, w.re, -nm3.re),
                                         m2.im + fma(q, w.im, -nm3.im)});
  const R n5 = c_norm(c5);
  if (!(c_norm(c4) <= R(1e6) * n5)) return false;
  const cx<R> t = c_mul(c_mul(c_mul(z[0], z[1]), z[2]), c5);  // -c5 z0 z1 z2
  const R nt = c_norm(t);
  const R ip = rcp_acc(n5 * nt);
  const R i5 = nt * ip, it = n5 * ip * (d * d);
  // S = z3 + z4 = c4/(-c5) - z0 - z1 - z2, P = z3 z4 = c0/(-c5 z0 z1 z2)
  const cx<R> S = {fma(fma(c4.re, c5.re, c4.im * c5.im), i5, -z[0].re) - z[1].re - z[2].re,
                   fma(fma(c4.im, c5.re, -c4.re * c5.im), i5, -z[0].im) - z[1].im - z[2].im};
  const cx<R> P = {fma(zeta.re, t.re, zeta.im * t.im) * it,
                   fma(zeta.im, t.re, -zeta.re * t.im) * it};
  const cx<R> hs = {R(0.5) * S.re, R(0.5) * S.im};
  const cx<R> D2 = c_fma(hs, hs, cx<R>{-P.re, -P.im});
  const R m = sqrt_acc(c_norm(D2));
  const R u = sqrt_acc(R(0.5) * (m + fabs(D2.re)));
  const R v = R(0.5) * D2.im * rcp_acc(u);
  const bool pos = !(D2.re < R(0.0));
  const cx<R> D = {pos ? u : v, pos ? v : u};  // (for re < 0: i (u - i v))
  z3 = {hs.re + D.re, hs.im + D.im};
  z4 = {hs.re - D.re, hs.im - D.im};
  return m > R(1e-8) * c_norm(hs);
}

// ---------------------------------------------------------------- fit

// Square-root-free Givens state for columns (1, A | y): D = diag(d1, d2),
// unit upper-triangular factor with off-diagonal r12, transformed right-hand
// side (t1, t2) and the accumulated weighted residual sum of squares.
template <typename R>
struct LsqT {
  R d1, d2, r12, t1, t2, sse;
};

// Include the row (x1, x2 | y) with weight w (Gentleman's algorithm).
template <typename R>
SBLM_FN void lsq_include(LsqT<R>& s, R w, R x1, R x2, R y) {
  if (w == R(0.0)) return;
  if (x1 != R(0.0)) {
    const R wx = w * x1;
    const R dp = fma(wx, x1, s.d1);
    const R r = rcp_acc(dp);
    const R cb = s.d1 * r, sb = wx * r;
    w = cb * w;
    s.d1 = dp;
    const R xk = x2;
    x2 = fma(-x1, s.r12, xk);
    s.r12 = fma(cb, s.r12, sb * xk);
    const R yk = y;
    y = fma(-x1, s.t1, yk);
    s.t1 = fma(cb, s.t1, sb * yk);
  }
  if (w == R(0.0)) return;
  if (x2 != R(0.0)) {
    const R wx = w * x2;
    const R dp = fma(wx, x2, s.d2);
    const R r = rcp_acc(dp);
    const R cb = s.d2 * r, sb = wx * r;
    w = cb * w;
    s.d2 = dp;
    const R yk = y;
    y = fma(-x2, s.t2, yk);
    s.t2 = fma(cb, s.t2, sb * yk);
  }
  s.sse = fma(w * y, y, s.sse);
}

// ---------------------------------------------------------------- warm start

// Weights (w1, w2, w3) of the roots of the three previous epochs t1 > t2 >
// t3 for the start at epoch t: quadratic (Lagrange in t) extrapolation when
// all three are known (have3), however far t lies beyond them; else linear
// from two (have2), scaled by the ratio of epoch spacings clamped to [0, 4];
// else the previous roots themselves.  Across a gap in the cadence (a night
// between two runs of epochs minutes apart) the root paths are smooth, and
// the curvature the three close epochs give carries the start to within one
// sweep, where the linear start, clamped, left most such epochs two or three
// sweeps short; a poor start over a very long gap costs sweeps, or a cold
// retry, never a wrong root.
template <typename R>
SBLM_FN void warm_weights(R t, R t1, R t2, R t3, bool have2, bool have3, R& w1, R& w2, R& w3) {
  w1 = R(1.0);
  w2 = R(0.0);
  w3 = R(0.0);
  const R d12 = t1 - t2, d23 = t2 - t3, d13 = t1 - t3;
  if (have2 && have3 && d12 > R(0.0) && d23 > R(0.0)) {
    const R a1 = t - t1, a2 = t - t2, a3 = t - t3;
    const R r = rcp_fast(d12 * d13 * d23);
    w1 = a2 * a3 * (d23 * r);
    w2 = -a1 * a3 * (d13 * r);
    w3 = a1 * a2 * (d12 * r);
  } else if (have2 && d12 > R(0.0)) {
    const R r = vmin(vmax((t - t1) * rcp_fast(d12), R(0.0)), R(4.0));
    w1 = R(1.0) + r;
    w2 = -r;
  }
}

// The start of one root at the new epoch from its values at the three
// previous epochs, with the weights of warm_weights.
template <typename R>
SBLM_FN cx<R> extrapolate(cx<R> z1, cx<R> z2, cx<R> z3, R w1, R w2, R w3) {
  return {fma(w1, z1.re, fma(w2, z2.re, w3 * z3.re)), fma(w1, z1.im, fma(w2, z2.im, w3 * z3.im))};
}

// ---------------------------------------------------------------- prediction

// Velocity of an image, dz/dt = (v - g conj(v)) inv with v = dzeta/dt, from g
// and inv = 1/(1 - |g|^2) at the image.
template <typename R>
SBLM_FN cx<R> image_velocity(cx<R> v, cx<R> g, R inv) {
  const cx<R> gv = c_mul(g, cx<R>{v.re, -v.im});
  return {(v.re - gv.re) * inv, (v.im - gv.im) * inv};
}

// An image z of a source at zeta with constant velocity vz: its velocity v
// and, from the expansion to third order in time, where it was and how fast it
// went a time h earlier (z2, v2) -- the history of a chain that starts here.
// Differentiating dz/dt + g conj(dz/dt) = vz, with h1 = dg/dconj(z) = 2 q b^3 -
// 2 a^3 and h2 = 6 (a^4 + q b^4), gives every order by the solve of
// image_velocity.
template <typename R>
SBLM_FN void image_history(cx<R> z, cx<R> zeta, cx<R> vz, R d, R q, R h, cx<R>& v, cx<R>& z2,
                           cx<R>& v2) {
  const LensAt<R> e = lens_at<true>(z, zeta, d, q);
  const R inv = rcp_acc(R(1.0) - c_norm(e.g));
  v = image_velocity(vz, e.g, inv);
  const cx<R> a3 = c_mul(e.a2, e.a), qb3 = c_mul(e.qb2, e.b);
  const cx<R> h1 = {R(2.0) * (qb3.re - a3.re), R(2.0) * (qb3.im - a3.im)};
  const cx<R> vb = {v.re, -v.im};
  const cx<R> gd = c_mul(h1, vb);  // dg/dt
  const cx<R> wa = c_mul(gd, vb);
  const cx<R> acc = image_velocity(cx<R>{-wa.re, -wa.im}, e.g, inv);
  const cx<R> ab = {acc.re, -acc.im};
  const cx<R> h2 = c_fma(e.a2, e.a2, c_mul(qb3, e.b));
  const cx<R> gdd = c_fma(h1, ab, c_mul(c_mul(cx<R>{R(6.0) * h2.re, R(6.0) * h2.im}, vb), vb));
  const cx<R> wj = c_fma(gdd, vb, c_mul(cx<R>{R(2.0) * gd.re, R(2.0) * gd.im}, ab));
  const cx<R> jerk = image_velocity(cx<R>{-wj.re, -wj.im}, e.g, inv);
  const R hh = R(0.5) * h, h3 = h * R(1.0 / 3.0);
  z2 = {fma(-h, fma(-hh, fma(-h3, jerk.re, acc.re), v.re), z.re),
        fma(-h, fma(-hh, fma(-h3, jerk.im, acc.im), v.im), z.im)};
  v2 = {fma(-h, fma(-hh, jerk.re, acc.re), v.re), fma(-h, fma(-hh, jerk.im, acc.im), v.im)};
}

// Weights for the position of an image at epoch t from its positions and
// velocities at the two previous epochs t1 > t2 (cubic Hermite extrapolation),
// z = z1 + wd (z1 - z2) + w1 v1 + w2 v2; along its velocity where t1 = t2.  The
// error is s^2 (s + h)^2 z^(4)/24 (s = t - t1, h = t1 - t2) against s (s + h)
// (s + 2h) z^(3)/6 for the parabola through three positions; it carries
// across a gap in the cadence (a night between two runs of epochs minutes
// apart) up to a thousand spacings, where rounding (about 2 (s/h)^3 ulp) takes
// over.  A poor start costs steps: what image_close accepts is an image.
template <typename R>
SBLM_FN void track_weights(R t, R t1, R t2, R& wd, R& w1, R& w2) {
  const R s = t - t1, h = t1 - t2;
  R r = s * rcp_fast(h);
  if (!(h > R(0.0) && r <= R(1e3))) r = R(0.0);
  const R u = R(1.0) + r;
  wd = r * r * fma(R(2.0), r, R(3.0));
  w1 = s * u * u;
  w2 = s * r * u;
  wd = -wd;
}

template <typename R>
SBLM_FN cx<R> predict(cx<R> z1, cx<R> z2, cx<R> v1, cx<R> v2, R wd, R w1, R w2) {
  return {fma(w1, v1.re, fma(w2, v2.re, fma(wd, z1.re - z2.re, z1.re))),
          fma(w1, v1.im, fma(w2, v2.im, fma(wd, z1.im - z2.im, z1.im)))};
}

}  // namespace sblm
