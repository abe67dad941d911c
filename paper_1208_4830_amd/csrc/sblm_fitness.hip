// sblm_fitness.hip -- batched binary-lens magnification and chi^2 fitness on
// gfx950 (MI355X).
//
// Method (Rajpaul 2012, Sec. 2.2 and Sec. 4): for every (individual, epoch)
// pair the source position follows Eq. (sourcePos) with tau = (t - t0)/tE;
// the images solve the lens equation Eq. (lensing), whose fifth-order
// polynomial form Eq. (lensingPoly) is solved here for all five roots; the
// two spurious roots are rejected by substitution into the lens equation;
// the magnification is sum_i 1/|det J_i| with
// det J = 1 - |1/conj(z)^2 + q/(d - conj(z))^2|^2.  The fitness is chi^2 of
// the blended flux Fs*A + Fb (Sec. 4.4, Eq. blend) with Fs, Fb profiled by
// weighted linear least squares.
//
// Mapping onto CDNA4:
//   * one group of G lanes per individual (8 to 64, several waves up to 256;
//     magnifications from 1 to as many as there are epochs), each lane owning
//     a contiguous chunk of C = ceil(L/G) epochs; the individual's parameters
//     are wave-uniform (scalar registers), epochs are read once;
//   * at the first epoch of a chunk all five roots are found together by the
//     Ehrlich-Aberth simultaneous iteration -- branch-free and identical work
//     per lane, so a wavefront stays in lockstep -- from the roots in the
//     limit of a light secondary.  The loop ends when every lane of the wave
//     has converged (wave vote);
//   * from there three images are followed on the lens equation itself, and
//     the other two roots, and with them the image count, come from the sum
//     and the product of all five (track_images); only an epoch that fails a
//     check there goes through the iteration again;
//   * FP64 mode iterates in FP64.  MIXED mode iterates in FP32 to a loose
//     tolerance, then continues in FP64 (normally two sweeps) from there; the
//     tracking, the image test, det J and the fit are FP64 in both modes;
//   * the weighted least-squares fit is accumulated on the fly with
//     square-root-free Givens rotations (Gentleman 1973, the row-update form
//     of a QR factorisation) over columns (1, A | y), so chi^2 comes out as
//     the accumulated residual, with no A stored and no cancellation of
//     large sums; lane results are merged by a fixed shuffle tree (bitwise
//     deterministic).
#include <math.h>
#include <stdarg.h>
#include <stdio.h>

#include "sblm_internal.h"

// Stopping tolerance of the FP64 root iteration: the estimated error left in
// every root after the last step, relative to max(1, |z|).  The roots only
// start the images: an accepted image whose residual on the lens equation
// could move A by more than 1e-12 relative is refined on the lens equation
// itself (see magnification), so this tolerance sets the work, not the
// accuracy of A: 1e-9 leaves the measured magnification errors as they are
// at 1e-16 (they first grow at 1e-8) while most warm-started solves end
// after one sweep.
#ifndef SBLM_ROOT_TAU
#define SBLM_ROOT_TAU 1e-9
#endif
// The FP32 iteration of the precision form only has to bring the roots
// within reach of two FP64 Newton steps (quadratic: an error e0 goes to
// about e0^2/s, then e0^4/s^3): an estimated error of 1e-5 relative.
#ifndef SBLM_ROOT_TAU32
#define SBLM_ROOT_TAU32 1e-5f
#endif

// Passes of track_images over images that are not final after their second
// step.
#define SBLM_TRACK_PASSES 8

namespace sblm {

// The primitive operations the shared arithmetic (sblm_math.h) takes from
// its number type, for FP64 and FP32 on the device.
// Smaller / larger of two values, the non-NaN one if one is NaN (one v_min /
// v_max where the operands are results of arithmetic, which the compiler knows
// to be quiet).
__device__ __forceinline__ double vmin(double a, double b) { return fmin(a, b); }
__device__ __forceinline__ float vmin(float a, float b) { return fminf(a, b); }
__device__ __forceinline__ double vmax(double a, double b) { return fmax(a, b); }
__device__ __forceinline__ float vmax(float a, float b) { return fmaxf(a, b); }
// Hardware reciprocal estimate (relative error < 5e-8 in FP64).
__device__ __forceinline__ double rcp_hw(double x) { return __builtin_amdgcn_rcp(x); }
__device__ __forceinline__ float rcp_hw(float x) { return __builtin_amdgcn_rcpf(x); }
// Hardware estimate of 1/sqrt(x) (relative error < 1e-7 in FP64).
__device__ __forceinline__ double rsq_hw(double x) { return __builtin_amdgcn_rsq(x); }

}  // namespace sblm

#include "sblm_math.h"

namespace sblm {

// Starting points for a cold solve from the limit of a light secondary
// (float, all lanes the same work).  At q = 0 the lens polynomial factors:
// the two images z+- of the primary alone, zeta (1 +- sqrt(1 + 4/|zeta|^2))/2,
// the spurious root 1/(d - conj(zeta)) and a double root at z = d; to first
// order in q the double root splits into z = d + q d u with
//   B u^2 + C u + E = 0,  E = zeta - d,  a = 1 + d conj(zeta),  b = a - d^2,
//   B = b (E a + d),  C = E (a + b) + d.
// Each start is turned by 1e-4 about the origin: starts on a common symmetry
// axis could otherwise leave it by rounding only.  Over the prior they take
// the iteration 2.7 sweeps per solve (7.6 for the slowest of 64), the circle
// of cold_start 7.8 (12.9); the roots reached are the same.  False when a
// start is not finite or two of them (nearly) coincide: then the circle.
__device__ __forceinline__ bool light_secondary_start(cx<double> zeta_, double d_, double q_,
                                                      cx<float> z[5]) {
  const float d = (float)d_, q = (float)q_;
  const cx<float> zt = {(float)zeta_.re, (float)zeta_.im};
  const float n = c_norm(zt);
  const float h = 0.5f + 0.5f * __builtin_amdgcn_sqrtf(fmaf(4.0f, rcp_hw(n), 1.0f));
  const float m = -rcp_hw(n * h);  // z- = -zeta/(|zeta|^2 h)
  z[0] = {h * zt.re, h * zt.im};
  z[1] = {m * zt.re, m * zt.im};
  const cx<float> E = {zt.re - d, zt.im};
  const float ie = rcp_hw(c_norm(E));  // d - conj(zeta) = -conj(E)
  z[2] = {-E.re * ie, -E.im * ie};
  const cx<float> a = {fmaf(d, zt.re, 1.0f), -d * zt.im};
  const cx<float> b = {fmaf(-d, d, a.re), a.im};
  const cx<float> Ea = c_mul(E, a);
  const cx<float> B = c_mul(b, cx<float>{Ea.re + d, Ea.im});
  const cx<float> Eab = c_fma(E, b, Ea);
  const cx<float> C = {Eab.re + d, Eab.im};
  // s = sqrt(C^2 - 4 B E), its sign such that C + s is the larger sum;
  // u = w/B and E/w with w = -(C + s)/2
  const cx<float> C2 = c_mul(C, C), BE = c_mul(B, E);
  const cx<float> D = {fmaf(-4.0f, BE.re, C2.re), fmaf(-4.0f, BE.im, C2.im)};
  const float r = __builtin_amdgcn_sqrtf(c_norm(D));
  const float t = __builtin_amdgcn_sqrtf(0.5f * (r + fabsf(D.re)));
  const float o = t > 0.0f ? 0.5f * D.im * rcp_hw(t) : 0.0f;
  cx<float> s = D.re >= 0.0f ? cx<float>{t, o} : cx<float>{fabsf(o), copysignf(t, D.im)};
  if (fmaf(C.re, s.re, C.im * s.im) < 0.0f) s = {-s.re, -s.im};
  const cx<float> w = {-0.5f * (C.re + s.re), -0.5f * (C.im + s.im)};
  const float qd = q * d;
  const float fb = qd * rcp_hw(c_norm(B)), fw = qd * rcp_hw(c_norm(w));
  z[3] = {fmaf(fb, fmaf(w.re, B.re, w.im * B.im), d), fb * fmaf(w.im, B.re, -w.re * B.im)};
  z[4] = {fmaf(fw, fmaf(E.re, w.re, E.im * w.im), d), fw * fmaf(E.im, w.re, -E.re * w.im)};
  const float turn[5] = {1e-4f, -0.7e-4f, 0.8e-4f, 1.3e-4f, -1.1e-4f};
  float sum = 0.0f, dmin = INFINITY;
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    z[i] = {fmaf(-turn[i], z[i].im, z[i].re), fmaf(turn[i], z[i].re, z[i].im)};
    sum += fabsf(z[i].re) + fabsf(z[i].im);
#pragma unroll
    for (int j = 0; j < i; ++j) dmin = vmin(c_norm(c_sub(z[i], z[j])), dmin);
  }
  return sum < 1e12f && dmin > 1e-12f;
}

// Starting points for a cold solve of the polynomial c of the source zeta and
// the lens d, q: those of the light-secondary limit where they apply (q <= 2,
// checked up to there), else five points on a circle about the root
// centroid -c4/(5 c5) of radius (|c0|/|c5|)^(1/5) (geometric mean of the
// root moduli); for a degree-4 polynomial four points and one root parked
// far away, where it never moves; with a far root (far_root) the four near
// roots start as for the degree-4 polynomial and the fifth at -c4/c5, which
// it would otherwise take the iteration some 50-80 sweeps to walk out to.
template <typename T>
__device__ __forceinline__ void cold_start(const cx<T> c[6], cx<double> zeta, double d, double q,
                                           bool deg4, cx<T> z[5], bool far = false) {
  const bool four = deg4 || far;
  if (!four && q <= 2.0) {
    cx<float> zf[5];
    if (light_secondary_start(zeta, d, q, zf)) {
#pragma unroll
      for (int i = 0; i < 5; ++i) z[i] = {(T)zf[i].re, (T)zf[i].im};
      return;
    }
  }
  // cos/sin of 2 pi k/5 + 0.4 and 2 pi k/4 + 0.4
  const float c5a[5] = {0.92106099f, 0.06083749f, -0.88523008f, -0.62472004f,
                        0.52805164f};
  const float s5a[5] = {0.38941834f, 0.99814771f, 0.46517413f, -0.78084257f,
                        -0.84920782f};
  const float c4a[4] = {0.92106099f, -0.38941834f, -0.92106099f, 0.38941834f};
  const float s4a[4] = {0.38941834f, 0.92106099f, -0.38941834f, -0.92106099f};
  const int lead = four ? 4 : 5;
  const float n_lead = (float)c_norm(c[lead]);
  const float n_0 = (float)c_norm(c[0]);
  float ratio = n_0 / n_lead;
  if (!(ratio > 1e-30f) || !(ratio < 1e30f)) ratio = 1.0f;
  const float R = powf(ratio, four ? 0.125f : 0.1f);
  // centroid = -c[lead-1] / (lead c[lead])
  const cx<float> a = {(float)c[lead - 1].re, (float)c[lead - 1].im};
  const cx<float> b = {(float)c[lead].re, (float)c[lead].im};
  const float ib = 1.0f / (fmaf(b.re, b.re, b.im * b.im) * (float)lead);
  const float cen_re = -(a.re * b.re + a.im * b.im) * ib;
  const float cen_im = -(a.im * b.re - a.re * b.im) * ib;
  if (four) {
#pragma unroll
    for (int k = 0; k < 4; ++k)
      z[k] = {(T)(cen_re + R * c4a[k]), (T)(cen_im + R * s4a[k])};
    z[4] = {(T)1e18, (T)1e18};
    if (far) {  // -c4/c5
      const T n5 = c_norm(c[5]);
      z[4] = {-(c[4].re * c[5].re + c[4].im * c[5].im) / n5,
              -(c[4].im * c[5].re - c[4].re * c[5].im) / n5};
    }
  } else {
#pragma unroll
    for (int k = 0; k < 5; ++k)
      z[k] = {(T)(cen_re + R * c5a[k]), (T)(cen_im + R * s5a[k])};
  }
}

// Images, det J and the magnification from five FP64 roots.  The image count
// and the choice of images use the roots' residuals (image_score), or where those
// tell no three images apart the distances that they stand for; an
// accepted image that needs it is refined on the lens equation
// (refine_image).  If next, *order receives, per root, its place when the three
// images to be tracked from here come first: with three images those, with five the
// three of largest |det J| (a pair about to merge goes last).  Returns A.
__device__ __forceinline__ double magnification(const cx<double> z[5],
                                                cx<double> zeta, double d,
                                                double q, bool deg4,
                                                int& nimg, int& npolish, bool next, int* order) {
  double r2[5], adet[5];
  bool refine[5];
#pragma unroll
  for (int i = 0; i < 5; ++i) refine[i] = image_score(z[i], zeta, d, q, &r2[i], &adet[i]);
  if (deg4) r2[4] = INFINITY;
  int below = 0;
#pragma unroll
  for (int i = 0; i < 5; ++i) below += (r2[i] < SBLM_IMAGE_TOL2) ? 1 : 0;
  const bool five = !deg4 && below >= 4;
  // Fewer than three roots that solve the lens equation to its tolerance: next to
  // a lens, in a cluster of roots (a separation below 3e-3, a mass ratio below
  // 1e-6), a root's rounding is a large residual, |g| times its distance to the
  // image.  There the distances are what is compared (not for a heavy secondary,
  // in whose units the clusters are the smaller and the other images the wider).
  if (below < 3 && q <= 2.0) {
#pragma unroll
    for (int i = 0; i < 5; ++i) r2[i] *= rcp_fast(1.0 + adet[i]);
  }
  // accepted images: sum those that need no refinement, list the others
  double A = 0.0;
  unsigned int todo = 0u;
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    int rank = 0;
#pragma unroll
    for (int j = 0; j < 5; ++j)
      rank += (r2[j] < r2[i] || (r2[j] == r2[i] && j < i)) ? 1 : 0;
    const bool acc = five || rank < 3;
    order[i] = rank;
    if (acc && refine[i])
      todo |= 1u << i;
    else if (acc)
      A += rcp_acc(adet[i]);
  }
  if (next && five) {
#pragma unroll
    for (int i = 0; i < 5; ++i) {
      int far = 0;
#pragma unroll
      for (int j = 0; j < 5; ++j)
        far += (adet[j] > adet[i] || (adet[j] == adet[i] && j < i)) ? 1 : 0;
      order[i] = far;
    }
  }
  // refinement: one image per lane per pass, so the wavefront runs as many
  // passes as the lane with the most images to refine
  while (__any(todo != 0u)) {
    if (todo) {
      const int i = __builtin_ctz(todo);
      todo &= todo - 1u;
      cx<double> zi = z[0];
#pragma unroll
      for (int k = 1; k < 5; ++k)
        if (i == k) zi = z[k];
      ++npolish;
      A += refine_image(zi, zeta, d, q);
    }
  }
  nimg = five ? 5 : 3;
  return A;
}

// The tracked form of an epoch: the three images predicted in z, stepped
// twice on the lens equation (a Newton step, then one that is judged), a lane's
// images that are not final yet one per pass after that; their velocities v
// for the source's vz; the other two roots from those.  True with A and the
// image count when every check holds (see sblm_math.h): the images final and
// apart, the other two roots clearly both images or clearly neither.
//   Over the batched set 98.4% of the epochs end here (1.6% are the first of
// a chain); in 95% of a wave's steps no lane is left for the iteration.
__device__ __forceinline__ bool track_images(cx<double> z[3], cx<double> v[3], cx<double> zeta,
                                             cx<double> vz, double d, double q, double& A,
                                             int& nimg, int passes = SBLM_TRACK_PASSES) {
  double ai[3];
  unsigned int todo = 0u;
#pragma unroll
  for (int i = 0; i < 3; ++i) image_newton(z[i], zeta, d, q);
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    cx<double> g;
    double inv;
    if (!image_close(z[i], zeta, d, q, &g, &inv)) todo |= 1u << i;
    ai[i] = fabs(inv);
    v[i] = image_velocity(vz, g, inv);
  }
  for (int pass = 0; pass < passes && __any(todo != 0u); ++pass) {
    if (todo) {
      const int i = __builtin_ctz(todo);
      cx<double> zi = i == 0 ? z[0] : i == 1 ? z[1] : z[2], g;
      double inv;
      const bool done = image_close(zi, zeta, d, q, &g, &inv);
      const cx<double> vi = image_velocity(vz, g, inv);
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if (i == k) {
          z[k] = zi;
          v[k] = vi;
          ai[k] = fabs(inv);
        }
      if (done) todo &= todo - 1u;
    }
  }
  A = ai[0] + ai[1] + ai[2];
  nimg = 3;
  double apart = c_norm(c_sub(z[0], z[1]));
  apart = vmin(c_norm(c_sub(z[0], z[2])), apart);
  apart = vmin(c_norm(c_sub(z[1], z[2])), apart);
  bool ok = todo == 0u && apart > SBLM_TRACK_APART2;
  cx<double> z3, z4;
  ok = other_roots(zeta, d, q, z, z3, z4) && ok;
  const double r3 = lens_residual2(z3, zeta, d, q), r4 = lens_residual2(z4, zeta, d, q);
  const bool spurious = r3 > SBLM_TRACK_SPURIOUS2 && r4 > SBLM_TRACK_SPURIOUS2;
  if (ok && !spurious) {  // five images?
    double i3, i4;
    cx<double> a = z3, b = z4, g;
    ok = r3 < SBLM_TRACK_IMAGE2 && r4 < SBLM_TRACK_IMAGE2;
    ok = image_close(a, zeta, d, q, &g, &i3) && ok;
    ok = image_close(b, zeta, d, q, &g, &i4) && ok;
    A += fabs(i3) + fabs(i4);
    nimg = 5;
  }
  return ok;
}

// ---------------------------------------------------------------- fit

using Lsq = LsqT<double>;

// ---------------------------------------------------------------- kernel

template <int G>
__device__ __forceinline__ double grp_shfl_down(double v, int off) {
  return __shfl_down(v, off, G);
}

// Per-lane counters (32 bits: a lane's share of one launch stays far below
// 2^32 events), summed over the wave and added to sblm_stats at the end.
struct LaneStats {
  unsigned int solves, iters, capped, fallback, deg4, wave_iters, iters32, polished, retried,
      unsettled, newton;
};
__device__ __forceinline__ void add_stats(LaneStats& a, const LaneStats& b) {
  a.solves += b.solves;
  a.iters += b.iters;
  a.capped += b.capped;
  a.fallback += b.fallback;
  a.deg4 += b.deg4;
  a.wave_iters += b.wave_iters;
  a.iters32 += b.iters32;
  a.polished += b.polished;
  a.retried += b.retried;
  a.unsettled += b.unsettled;
  a.newton += b.newton;
}
// ... and, in MIXED, the epochs tracked (in FP64, which has no polish passes,
// those are `newton`: one more register through the loops costs spills).
struct WaveStats : LaneStats {
  unsigned int tracked;
};

// A solve that reaches the iteration cap has settled when its roots are
// finite and its last sweep moved them by less than this much relative
// (squared, i.e. 1e-4): the iteration has stalled at the rounding level next
// to a near-multiple root -- two images merging at a fold of the caustic,
// three at a cusp, where FP64 resolves the roots only to about eps^(1/2) and
// eps^(1/3) ~ 6e-6 relative and the steps jitter at that level; the
// accepted images are refined on the lens equation anyway.
#define SBLM_SETTLED_STEP2 1e-8

// Solve one polynomial (of the source zeta and the lens d, q) from the roots
// in z (warm) or from a cold start;
// ok = converged to finite roots; settled = ok, or capped with finite roots
// that no longer move (see SBLM_SETTLED_STEP2).  `retry` marks a second,
// cold attempt at an epoch whose warm-started solve failed (not counted as
// another solve).
template <int MODE>
__device__ __forceinline__ void solve_roots(const cx<double> c[6], cx<double> zeta, double d,
                                            double q, bool deg4, bool warm, bool active,
                                            cx<double> z[5], LaneStats& st,
                                            bool& ok, bool& settled, bool retry = false) {
  constexpr int MAXIT64 = 60, MAXIT32 = 30;
  // estimated relative error left after the last step
  const double tau64 = SBLM_ROOT_TAU;
  const float tau32 = SBLM_ROOT_TAU32;
  const bool far = !deg4 && far_root(c);
  if (!warm && active) cold_start<double>(c, zeta, d, q, deg4, z, far);
  unsigned int it_lane = 0, it32_lane = 0, it_wave = 0, newton_lane = 0;
  bool done = !active, fell_back = false;
  if (MODE == SBLM_MIXED) {
    // The precision form: the root iteration in FP32 to a loose tolerance,
    // then at most two FP64 Newton steps on every root, the image test, det J
    // and the fit in FP64.  A polish that has not converged after two steps
    // falls back to FP64 Aberth sweeps from the polished roots (counted).
    // A warm start (the previous epochs' roots, extrapolated) is already as
    // close as FP32 can resolve and goes straight to the polish; degree-4
    // polynomials (parked root out of FP32 range) and those with a far root
    // (its powers overflow FP32) straight to FP64 sweeps.  The FP32
    // iteration ends at its own convergence test, or, after its first few
    // sweeps (the global phase, where steps need not shrink), when its steps
    // stop shrinking (the FP32 rounding floor next to clustered roots).
    const bool use32 = !deg4 && !far;
    cx<float> cf[6];
#pragma unroll
    for (int j = 0; j < 6; ++j) cf[j] = {(float)c[j].re, (float)c[j].im};
    cx<float> zf[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) zf[i] = {(float)z[i].re, (float)z[i].im};
    bool done32 = done || !use32 || warm;
    float prev = INFINITY;
    for (int it = 0; it < MAXIT32; ++it) {
      if (__all(done32)) break;
      ++it_wave;
      if (!done32) {
        float em;
        done32 = aberth_sweep<true>(cf, zf, false, tau32, &em);
        done32 = done32 || (it >= 4 && em > 0.25f * prev);  // shrank by < 2x
        prev = em;
        ++it32_lane;
      }
    }
    const bool polish = active && use32;
    if (polish && !warm) {
#pragma unroll
      for (int i = 0; i < 5; ++i) z[i] = {(double)zf[i].re, (double)zf[i].im};
    }
    double d2[5];
    nearest2(z, d2);
    bool pol_done = !polish;
    for (int k = 0; k < 2; ++k) {
      if (__all(pol_done)) break;
      ++it_wave;
      if (!pol_done) {
        pol_done = newton_pass(c, z, d2, tau64);
        ++newton_lane;
      }
    }
    if (polish) {
      // Newton steps that drew two roots together (a root taken over by its
      // neighbour's basin) leave the distinct FP32 roots behind: start the
      // FP64 iteration afresh
      double d2n[5];
      nearest2(z, d2n);
      bool apart = true;
#pragma unroll
      for (int i = 0; i < 5; ++i) apart = apart && (d2n[i] >= 0.25 * d2[i]);
      if (!apart) cold_start<double>(c, zeta, d, q, deg4, z, far);
      done = pol_done && apart;
      fell_back = !done;
    }
  }
  for (int it = 0; it < MAXIT64; ++it) {
    if (__all(done)) break;
    ++it_wave;
    if (!done) {
      done = aberth_sweep<false>(c, z, deg4, tau64, (double*)nullptr);
      ++it_lane;
    }
  }
  // a capped solve: one more sweep measures how far its roots still move
  double em_last = 0.0;
  if (__any(active && !done)) {
    if (active && !done) (void)aberth_sweep<true>(c, z, deg4, tau64, &em_last);
  }
  bool finite = true;
#pragma unroll
  for (int i = 0; i < 5; ++i)
    finite = finite && isfinite(z[i].re) && isfinite(z[i].im);
  ok = done && finite;
  settled = finite && (done || em_last <= SBLM_SETTLED_STEP2);
  if (active) {
    st.solves += retry ? 0 : 1;
    st.iters += it_lane + it32_lane;
    st.deg4 += (deg4 && !retry) ? 1 : 0;
    // MIXED: a polish that needed the FP64 iteration after its two steps
    if (MODE == SBLM_MIXED) st.fallback += fell_back ? 1 : 0;
    st.iters32 += it32_lane;
    st.newton += newton_lane;
  }
  st.wave_iters += it_wave;
}

// Per-lane context of one work item: the individual, its parameters and the
// lane's chunk [k0, k1) of the lightcurve's epochs.
struct Item {
  bool valid;
  int gl;  // lane within the group
  int64_t ind;
  double q, d, u0, sa, ca, t0, itE;
  int64_t e0, L, k0, k1, Cg;  // L: its epochs, Cg: the longest chunk
};

// The transcendental part of an individual's set-up: q = 10^(log10 q),
// sin and cos of alpha, 1/tE.  Out of line: inlined, the many constants of
// the exp10 and sincos expansions are hoisted out of the persistent grid's
// work loop into registers that then spill to scratch memory in every wave.
struct ItemTrig {
  double q, sa, ca, itE;
};
__device__ __noinline__ ItemTrig item_trig(double lq, double alpha, double tE) {
  ItemTrig r;
  r.q = exp10(lq);
  sincos(alpha, &r.sa, &r.ca);
  r.itE = 1.0 / tE;
  return r;
}

// Value of G for magnifications spread over any number of waves.
constexpr int WIDE = 1 << 20;

template <int G>
__device__ __forceinline__ Item item_setup(const FitArgs& a, int64_t wave_item) {
  Item x;
  const int lane = threadIdx.x & 63;
  int64_t item;
  int64_t lanes = G;
  if constexpr (G == WIDE) {  // as below, the number of waves set at run time
    lanes = a.lanes_per_ind;
    const int64_t parts = lanes / 64;
    item = wave_item / parts;
    x.gl = (int)(wave_item - item * parts) * 64 + lane;
  } else if constexpr (G > 64) {  // G / 64 waves per individual: wave item = (individual, part)
    item = wave_item / (G / 64);
    x.gl = (int)(wave_item % (G / 64)) * 64 + lane;
  } else {
    x.gl = lane & (G - 1);
    item = wave_item * (64 / G) + (lane / G);
  }
  x.valid = item < a.n_ind;
  x.ind = x.valid ? (a.order ? (int64_t)a.order[item] : item) : 0;
  // parameters of this individual (uniform within the group)
  double th[SBLM_NPAR];
#pragma unroll
  for (int j = 0; j < SBLM_NPAR; ++j) {
    const double v = x.valid ? a.theta[j * a.n_ind + x.ind] : 0.5;
    th[j] = a.encoded ? a.lo[j] + a.span[j] * v : v;
  }
  const ItemTrig tr = item_trig(th[0], th[3], th[4]);
  x.q = tr.q;
  x.d = th[1];
  x.u0 = th[2];
  x.t0 = th[5];
  x.sa = tr.sa;
  x.ca = tr.ca;
  x.itE = tr.itE;
  int64_t e0 = 0, e1 = a.n_t;
  if (a.off) {
    const int64_t lc = x.ind / a.pop;
    e0 = x.valid ? a.off[lc] : 0;
    e1 = x.valid ? a.off[lc + 1] : 0;
    if (a.skip && x.valid && a.skip[x.ind / a.skip_per]) e1 = e0;
  }
  if (!x.valid) e1 = e0;
  x.e0 = e0;
  const int64_t L = e1 - e0;
  x.L = L;
  x.Cg = (L + lanes - 1) / lanes;
  x.k0 = e0 + x.gl * x.Cg;
  x.k1 = (x.k0 + x.Cg < e1) ? x.k0 + x.Cg : e1;
  return x;
}

// Per-lane history, kept in LDS (touched once per epoch, at the prediction; in
// registers it would hold 24 or 40 VGPRs through the whole epoch).  Dynamic
// shared memory of ROOT_HIST_BYTES per thread; element [((slot*5 + i)*2 + part)
// * blockDim.x + thread] holds, real (part 0) or imaginary (part 1), of a
// tracked chain the position (slot 0) and the velocity (slot 1) of image i < 3
// at the previous epoch but one, else root i at that epoch (slot 0) and at the
// one before it (slot 1).
constexpr size_t ROOT_HIST_BYTES = 2 * 5 * 2 * sizeof(double);

// Dynamic shared memory: the root history, then (G > 64) one least-squares
// state per wave for the merge across the waves of an individual.
extern __shared__ double fit_dyn_smem[];

// Merge the lanes' least-squares states of each group (fixed tree) and write
// chi^2, Fs, Fb of the group's individual.  With G > 64 each wave merges its
// 64 lanes the same way, and the first wave of the individual then absorbs
// the states of the others in wave order (all waves of the block pass one
// barrier here).
template <int G>
__device__ __forceinline__ void finish_chi2(const FitArgs& a, const Item& x, Lsq ls) {
  constexpr int GW = G > 64 ? 64 : G;  // lanes merged by shuffles
  const int gl = x.gl;
  const bool valid = x.valid;
  const int64_t ind = x.ind;
  {
    // lane gl absorbs lane gl + off: fixed tree inside each group (wave)
#pragma unroll
    for (int off = GW / 2; off >= 1; off >>= 1) {
      Lsq o;
      o.d1 = grp_shfl_down<GW>(ls.d1, off);
      o.d2 = grp_shfl_down<GW>(ls.d2, off);
      o.r12 = grp_shfl_down<GW>(ls.r12, off);
      o.t1 = grp_shfl_down<GW>(ls.t1, off);
      o.t2 = grp_shfl_down<GW>(ls.t2, off);
      o.sse = grp_shfl_down<GW>(ls.sse, off);
      if ((gl & (GW - 1)) < off) {
        lsq_include(ls, o.d1, 1.0, o.r12, o.t1);
        lsq_include(ls, o.d2, 0.0, 1.0, o.t2);
        ls.sse += o.sse;
      }
    }
    if constexpr (G > 64) {
      double* part = fit_dyn_smem + (ROOT_HIST_BYTES / sizeof(double)) * blockDim.x;
      const int w = threadIdx.x >> 6;
      if ((threadIdx.x & 63) == 0) {
        part[w * 6 + 0] = ls.d1;
        part[w * 6 + 1] = ls.d2;
        part[w * 6 + 2] = ls.r12;
        part[w * 6 + 3] = ls.t1;
        part[w * 6 + 4] = ls.t2;
        part[w * 6 + 5] = ls.sse;
      }
      __syncthreads();
      if (gl == 0) {
        for (int p = 1; p < G / 64; ++p) {
          const double* o = part + (w + p) * 6;
          lsq_include(ls, o[0], 1.0, o[2], o[3]);
          lsq_include(ls, o[1], 0.0, 1.0, o[4]);
          ls.sse += o[5];
        }
      }
    }
    if (gl == 0 && valid) {
      const double saa = fma(ls.d1 * ls.r12, ls.r12, ls.d2);
      double fs, fb, c2;
      if (!(ls.d2 > 1e-14 * saa)) {  // singular 2x2 system
        fs = 0.0;
        fb = ls.t1;
        c2 = fma(ls.d2 * ls.t2, ls.t2, ls.sse);
      } else {
        fs = ls.t2;
        fb = fma(-ls.r12, fs, ls.t1);
        c2 = ls.sse;
      }
      a.chi2[ind] = c2;
      a.Fs[ind] = fs;
      a.Fb[ind] = fb;
      if (a.stats && !(ls.d2 > 1e-14 * saa))
        atomicAdd(&a.stats->n_degenerate, 1ull);
    }
  }

}

struct RootHist {
  double* h;
  __device__ __forceinline__ cx<double> get(int slot, int i) const {
    const int n = blockDim.x;
    return {h[((slot * 5 + i) * 2) * n + threadIdx.x],
            h[((slot * 5 + i) * 2 + 1) * n + threadIdx.x]};
  }
  __device__ __forceinline__ void set(int slot, int i, cx<double> v) const {
    const int n = blockDim.x;
    h[((slot * 5 + i) * 2) * n + threadIdx.x] = v.re;
    h[((slot * 5 + i) * 2 + 1) * n + threadIdx.x] = v.im;
  }
};

// Where a lane saves its first epoch's start for the next simplex round.
template <int G>
__device__ __forceinline__ double* root_cache_of(const FitArgs& a, const Item& x) {
  return a.root_cache ? a.root_cache + (x.ind * G + x.gl) * ROOT_CACHE : nullptr;
}

// Simplex rounds: a lane's first epoch starts from what the lane found there
// for the same trial slot in the previous round (the simplex moves little
// between rounds), else cold -- always cold in the first round of a run, so
// that a run does not depend on what ran in its slot before.  N roots or images.
template <int N>
__device__ __forceinline__ bool cached_start(const FitArgs& a, const Item& x, const double* rc,
                                             cx<double>* z) {
  if (a.cold && a.cold[x.ind / a.cold_per]) return false;
  cx<double> zc[N];
  bool fin = true;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    zc[i] = {rc[2 * i], rc[2 * i + 1]};
    fin = fin && isfinite(zc[i].re) && isfinite(zc[i].im);
  }
  if (fin) {
#pragma unroll
    for (int i = 0; i < N; ++i) z[i] = zc[i];
  }
  return fin;
}

template <int N>
__device__ __forceinline__ void save_start(double* rc, const cx<double>* z, bool ok) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    rc[2 * i] = ok ? z[i].re : NAN;
    rc[2 * i + 1] = ok ? z[i].im : NAN;
  }
}

// An epoch's magnification: a row of the fit, or the output.
template <bool CHI2>
__device__ __forceinline__ void put_epoch(const FitArgs& a, const Item& x, int64_t k, double wk,
                                          double yk, double A, int nimg, Lsq& ls) {
  if (CHI2) {
    lsq_include(ls, wk, 1.0, A, yk);
  } else {
    const int64_t o = x.ind * a.n_t + (k - x.e0);
    a.A[o] = A;
    if (a.n_img) a.n_img[o] = (int8_t)nimg;
  }
}

// The cold solve of an epoch whose images cannot be tracked, by the whole wave
// when any lane needs it (the others only follow along): the five roots by
// simultaneous iteration, the images and, where an epoch follows, which of
// them are tracked.  With SOLVE_RETRY the second attempt of a chain that is not
// tracked.  (A start from the images predicted and the two other roots they
// give takes more sweeps where those were no images: in simplex rounds, whose
// chains start from other parameters' images, 5.3 a solve against 2.3 cold, 18.8
// ms against 17.6 for 64 x 1000 epochs and 300 steps.)  Out of line: few steps
// come here, and inlined it costs the tracked form registers (64 x 1000 x 256
// FP64: 838 us inlined, 751 so).  out[0..9] receives the roots (SOLVE_NEXT: the
// images to track come first), out[10] A; flags in: SOLVE_ACTIVE, _NEXT, _RETRY,
// and _FOLLOW for a lane with an epoch that needs no solve; flags out: SOLVE_OK,
// the image count from bit 4; cnt: the lane's counters (added to).
enum {
  SOLVE_ACTIVE = 1,
  SOLVE_NEXT = 2,
  SOLVE_FOLLOW = 4,
  SOLVE_RETRY = 8,
  SOLVE_OK = 1
};
template <int MODE>
__device__ __noinline__ int solve_epoch(double zeta_re, double zeta_im, double d, double q,
                                        int flags, double* out, LaneStats* cnt) {
  const bool active = (flags & SOLVE_ACTIVE) != 0;
  const cx<double> zeta = {zeta_re, zeta_im};
  cx<double> z[5], c[6];
#pragma unroll
  for (int i = 0; i < 5; ++i) z[i] = {0.0, 0.0};
  lens_coeffs(zeta, d, q, c);
  const bool deg4 = drop_to_degree4(c);
  LaneStats st = {};
  bool ok, settled;
  solve_roots<MODE>(c, zeta, d, q, deg4, false, active, z, st, ok, settled,
                    (flags & SOLVE_RETRY) != 0);
  int r = 0;
  if (active) {
    int npol = 0, order[5], nimg;
    const bool next = (flags & SOLVE_NEXT) != 0;
    double A = magnification(z, zeta, d, q, deg4, nimg, npol, next, order);
    if (!settled) {  // (A and with it chi^2 become NaN, which ranks last)
      A = NAN;
      nimg = 0;
    }
    out[10] = A;
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      cx<double> zk = z[k];
      if (next) {
#pragma unroll
        for (int i = 0; i < 5; ++i)
          if (order[i] == k) zk = z[i];
      }
      out[2 * k] = zk.re;
      out[2 * k + 1] = zk.im;
    }
    r = (ok ? SOLVE_OK : 0) | (nimg << 4);
    cnt->solves += st.solves;
    cnt->iters += st.iters;
    cnt->capped += ok ? 0 : 1;
    cnt->fallback += st.fallback;
    cnt->deg4 += st.deg4;
    cnt->iters32 += st.iters32;
    cnt->polished += npol;
    cnt->unsettled += settled ? 0 : 1;
    cnt->newton += st.newton;
  }
  if (flags & (SOLVE_ACTIVE | SOLVE_FOLLOW)) cnt->wave_iters += st.wave_iters;
  return r;
}

// Chains that are solved at every epoch, Cg of them in this lane and at most C
// in the wave: the five roots start from those of the epochs before.
template <int MODE, bool CHI2, int G>
__device__ __forceinline__ void solve_chain(const FitArgs& a, const Item& x, int64_t Cg, int64_t C,
                                            LaneStats& st, Lsq& ls) {
  const int64_t k0 = x.k0, k1 = x.k1;
  const double q = x.q, d = x.d, t0 = x.t0;
  cx<double> z[5];
  const RootHist hist = {fit_dyn_smem};  // the roots one (slot 0) and two epochs before z
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    z[i] = {0.0, 0.0};
    hist.set(0, i, {0.0, 0.0});
    hist.set(1, i, {0.0, 0.0});
  }
  int nhist = 0;                        // epochs known
  double t1 = 0.0, t2 = 0.0, t3 = 0.0;  // those epochs

  // the epoch time one step ahead, the observation at the top of its step:
  // the loads are in flight during the solve
  double t_next = (0 < Cg && k0 < k1) ? a.t[k0] : t0;
  for (int64_t s = 0; s < C; ++s) {
    const int64_t k = k0 + s;
    const bool active = (s < Cg) && (k < k1);
    const double t = active ? t_next : t0;
    t_next = (s + 1 < Cg && k + 1 < k1) ? a.t[k + 1] : t0;
    double wk = 0.0, yk = 0.0;
    if (CHI2 && active) {
      wk = a.w[k];
      yk = a.y[k];
    }
    // the root history, read before the polynomial is formed (its latency
    // then overlaps the coefficients)
    cx<double> hp[5], hpp[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) {
      hp[i] = hist.get(0, i);
      hpp[i] = hist.get(1, i);
    }
    const cx<double> zeta = source_position(t, t0, x.itE, x.sa, x.ca, x.u0);
    cx<double> c[6];
    lens_coeffs(zeta, d, q, c);
    const bool deg4 = drop_to_degree4(c);
    bool cached = false;  // started from the root cache (not a solved epoch)
    double* rc = nullptr;
    if constexpr (CHI2 && G >= 64) {
      if (s == 0 && active) {
        rc = root_cache_of<G>(a, x);
        if (rc && !deg4) cached = cached_start<5>(a, x, rc, z);
      }
    }
    const bool warm = (nhist >= 1 || cached) && !deg4;
    // Warm start: quadratic (Lagrange in t) extrapolation of every root from
    // the three previous epochs, else linear from two (warm_weights); the
    // history shifts as it is used.
    {
      double w1, w2, w3;
      warm_weights(t, t1, t2, t3, nhist >= 2, nhist >= 3, w1, w2, w3);
#pragma unroll
      for (int i = 0; i < 5; ++i) {
        const cx<double> old = z[i];
        z[i] = extrapolate(old, hp[i], hpp[i], w1, w2, w3);
        hist.set(1, i, hp[i]);
        hist.set(0, i, old);
      }
    }
    bool ok, settled;
    const unsigned int w0 = st.wave_iters;
    solve_roots<MODE>(c, zeta, d, q, deg4, warm, active, z, st, ok, settled);
    if (!active) st.wave_iters = w0;
    // a warm start that did not converge: solve again from the cold start;
    // roots that still have not settled poison the result (A and with it chi^2
    // become NaN, which ranks last)
    const bool again = active && !ok && warm;
    double A = 0.0;
    int nimg = 0;
    if (__any(again)) {
      double io[11];
      LaneStats rs = {};
      const int out =
          solve_epoch<MODE>(zeta.re, zeta.im, d, q,
                            again ? SOLVE_ACTIVE | SOLVE_RETRY : active ? SOLVE_FOLLOW : 0, io,
                            &rs);
      if (again) {
        A = io[10];
        nimg = out >> 4;
        ok = (out & SOLVE_OK) != 0;
#pragma unroll
        for (int i = 0; i < 5; ++i) z[i] = {io[2 * i], io[2 * i + 1]};
        st.retried += 1;
      }
      add_stats(st, rs);
    }
    if constexpr (CHI2 && G >= 64) {
      if (rc) save_start<5>(rc, z, ok);
    }
    // (roots started from the cache follow no solved epoch, roots of a retry
    // are in another order, a degree-4 polynomial's are not those of the next:
    // the next epoch extrapolates from this one alone)
    nhist = (!ok || deg4) ? 0 : (warm && !cached && !again) ? (nhist < 3 ? nhist + 1 : 3) : 1;
    t3 = t2;
    t2 = t1;
    t1 = t;
    if (active) {
      if (!again) {
        int npol = 0, order[5];
        A = magnification(z, zeta, d, q, deg4, nimg, npol, false, order);
        st.polished += npol;
        st.capped += ok ? 0 : 1;
        if (!settled) {
          A = NAN;
          nimg = 0;
          st.unsettled += 1;
        }
      }
      put_epoch<CHI2>(a, x, k, wk, yk, A, nimg, ls);
    }
  }
}

// Chains along which three images are carried: predicted from the epochs
// before and tracked (track_images); the lanes that fail a check solve for all
// five roots (solve_epoch), which a wave goes through when any of its lanes
// does.
//   Bound by FP64 arithmetic (899 FLOPs per tracked epoch, 1920 of a solve with
// the sweeps a wave takes in lockstep).  Solved at every epoch, 256 x 1000
// epochs x 256 individuals took 4.23 ms FP64 over the prior and 3.23 ms for an
// evolved population, tracked 2.43 and 2.05; 256 x 200-5000 x 128 5.03 and 3.07
// ms; 64 x 1000 x 256 MIXED 1.58 and 0.83 ms.  The bound on the length of a judged
// step (image_close), not yet in these, costs 1.5%: 1.97 and 2.00 ms, 0.83 and 0.84.
template <int MODE, bool CHI2, int G>
__device__ __forceinline__ void track_chain(const FitArgs& a, const Item& x, int64_t Cg, int64_t C,
                                            WaveStats& st, Lsq& ls) {
  const int64_t k0 = x.k0, k1 = x.k1;
  const double q = x.q, d = x.d, t0 = x.t0;
  cx<double> zt[3], vt[3];  // the images at the epoch before, their velocities
  const RootHist hist = {fit_dyn_smem};  // ... at the one before that (slots 0 and 1)
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    zt[i] = {0.0, 0.0};
    vt[i] = {0.0, 0.0};
    hist.set(0, i, {0.0, 0.0});
    hist.set(1, i, {0.0, 0.0});
  }
  const cx<double> vz = {x.sa * x.itE, -x.ca * x.itE};  // the source's velocity
  bool warm = false;                                    // the images are known
  double t1 = 0.0, t2 = 0.0;                            // those epochs
  unsigned int tracked = 0;
  LaneStats slow = {};  // (in memory: solve_epoch adds to it)

  double t_next = (0 < Cg && k0 < k1) ? a.t[k0] : t0;  // as in solve_chain
  for (int64_t s = 0; s < C; ++s) {
    const int64_t k = k0 + s;
    const bool active = (s < Cg) && (k < k1);
    const double t = active ? t_next : t0;
    t_next = (s + 1 < Cg && k + 1 < k1) ? a.t[k + 1] : t0;
    double wk = 0.0, yk = 0.0;
    if (CHI2 && active) {
      wk = a.w[k];
      yk = a.y[k];
    }
    const cx<double> zeta = source_position(t, t0, x.itE, x.sa, x.ca, x.u0);
    double* rc = nullptr;
    if constexpr (CHI2 && G >= 64) {
      if (s == 0 && active) {
        rc = root_cache_of<G>(a, x);
        if (rc) warm = cached_start<3>(a, x, rc, zt);
      }
    }
    // prediction of every image (track_weights); the history shifts as it is
    // used
    {
      double wd, w1, w2;
      track_weights(t, t1, t2, wd, w1, w2);
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const cx<double> z1 = zt[i];
        zt[i] = predict(z1, hist.get(0, i), vt[i], hist.get(1, i), wd, w1, w2);
        hist.set(0, i, z1);
        hist.set(1, i, vt[i]);
      }
    }
    double A = 0.0;
    int nimg = 3;
    bool ok = true, need = active;
    if (active && warm) {
      need = !track_images(zt, vt, zeta, vz, d, q, A, nimg);
      tracked += need ? 0u : 1u;
    }
    const bool any_need = __any(need);
    if (any_need) {
      double io[11];
      const int out = solve_epoch<MODE>(
          zeta.re, zeta.im, d, q, need ? SOLVE_ACTIVE | SOLVE_NEXT : active ? SOLVE_FOLLOW : 0,
          io, &slow);
      if (need) {
        A = io[10];
        nimg = out >> 4;
        ok = (out & SOLVE_OK) != 0;
#pragma unroll
        for (int i = 0; i < 3; ++i) zt[i] = {io[2 * i], io[2 * i + 1]};
      }
    }
    if constexpr (CHI2 && G >= 64) {
      if (rc) save_start<3>(rc, zt, ok);
    }
    // a chain that starts here: its history from the expansion of the images
    // about this epoch
    if (s + 1 < C && (s == 0 || any_need)) {
      if (s == 0 || need) {
        const double h = t_next - t;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          cx<double> z2, v2;
          image_history(zt[i], zeta, vz, d, q, h, vt[i], z2, v2);
          hist.set(0, i, z2);
          hist.set(1, i, v2);
        }
        t1 = t - h;
      }
    }
    warm = ok;
    t2 = t1;
    t1 = t;
    if (active) put_epoch<CHI2>(a, x, k, wk, yk, A, nimg, ls);
  }
  slow.solves += tracked;
  slow.newton += tracked;
  if (MODE == SBLM_MIXED) st.tracked += tracked;
  add_stats(st, slow);
}

// The longest of the chunks c of a wave's groups.
template <int G>
__device__ __forceinline__ int64_t wave_longest(int64_t c) {
#pragma unroll
  for (int o = G; o < 64; o <<= 1) {
    const int64_t oc = __shfl_xor(c, o, 64);
    c = oc > c ? oc : c;
  }
  return c;
}

// One wave's share of the work: 64/G individuals (items wave_item*64/G ...);
// every lane takes its s-th epoch at the same time.  Where a wave holds chains
// of both kinds (tracked_chains, simplex_tracked) it goes through both loops.
template <int MODE, bool CHI2, int G>
__device__ __forceinline__ void fit_wave(const FitArgs& a, int64_t wave_item, WaveStats& st) {
  const Item x = item_setup<G>(a, wave_item);
  Lsq ls = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  const int64_t lanes = G == WIDE ? a.lanes_per_ind : G;
  const bool track =
      a.by_chain ? simplex_tracked(x.Cg) : tracked_chains(a.n_ind, lanes, x.L, x.Cg);
  const int64_t Cs = track ? 0 : x.Cg, Ct = track ? x.Cg : 0;
  const int64_t ws = wave_longest<G>(Cs), wt = wave_longest<G>(Ct);
  if (ws > 0) solve_chain<MODE, CHI2, G>(a, x, Cs, ws, st, ls);
  if (wt > 0) track_chain<MODE, CHI2, G>(a, x, Ct, wt, st, ls);
  if (CHI2) finish_chi2<G>(a, x, ls);
}

// Adds the wave's counters.
template <int MODE>
__device__ __forceinline__ void put_stats(sblm_stats* stats, const WaveStats& st, int lane) {
  // wave sums in 64 bits
  unsigned long long v[12] = {st.solves,     st.iters,   st.capped,   st.fallback,
                              st.deg4,       st.wave_iters, st.iters32, st.polished,
                              st.retried,    st.unsettled, st.newton,
                              MODE == SBLM_MIXED ? st.tracked : 0u};
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1)
#pragma unroll
    for (int k = 0; k < 12; ++k) v[k] += __shfl_down(v[k], off, 64);
  if (MODE != SBLM_MIXED) v[11] = v[10];
  if (lane == 0 && v[0]) {
    unsigned long long* dst[12] = {&stats->n_solves,    &stats->n_iter,
                                   &stats->n_capped,    &stats->n_fallback,
                                   &stats->n_degree4,   &stats->n_wave_iter,
                                   &stats->n_iter_fp32, &stats->n_polished,
                                   &stats->n_retried,   &stats->n_unsettled,
                                   &stats->n_newton,    &stats->n_tracked};
#pragma unroll
    for (int k = 0; k < 12; ++k)
      if (v[k]) atomicAdd(dst[k], v[k]);
  }
}

// PERSIST = 0: one-shot grid.  PERSIST = 1: persistent grid fed by a work
// counter.  All forms are compiled for two waves per SIMD: left alone, the
// mixed form takes 272 registers and runs one, where its dependent FP64
// chains leave the SIMD idle half of the time.
template <int MODE, bool CHI2, int G, int PERSIST>
__global__ __launch_bounds__(256, 2) void fitness_kernel(
    FitArgs a) {
  // (blocks of at most 256 threads: launch_gg refuses larger ones)
  constexpr int GPW = G > 64 ? 1 : 64 / G;  // individuals per wave
  const int lane = threadIdx.x & 63;
  WaveStats st = {};
  // One-shot grid: wave w takes wave item w (blocks remapped so that
  // consecutive logical blocks sit on one XCD, unless a work order is
  // given).  Persistent grid: waves take items from a shared counter until
  // it runs past the last one, so every wave reaches the exit.  One call
  // site keeps one inlined copy of the body.
  const int64_t n_wave_items = G > 64 ? a.n_ind * (G / 64) : (a.n_ind + GPW - 1) / GPW;
  if constexpr (PERSIST) {
    if (a.xcd_start) {
      // per-XCD queues: first the items of the lightcurves this block's XCD
      // owns (their epochs stay in its L2; workgroups are dealt to the XCDs
      // round-robin), then what is left in the other XCDs' queues.  Each
      // queue is visited until it runs past its last item, so every wave
      // reaches the exit.
      const int x0 = blockIdx.x & 7;
      for (int k = 0; k < 8; ++k) {
        const int x = (x0 + k) & 7;
        const int64_t w0 = (a.xcd_start[x] + GPW - 1) / GPW;
        const int64_t w1 = (a.xcd_start[x + 1] + GPW - 1) / GPW;
        for (;;) {
          unsigned int v = 0;
          if (lane == 0) v = atomicAdd(a.queue + x, 1u);
          const int64_t wi = w0 + (int64_t)__shfl(v, 0, 64);
          if (wi >= w1) break;
          fit_wave<MODE, CHI2, G>(a, wi, st);
        }
      }
    } else {
      for (;;) {
        unsigned int v = 0;
        if (lane == 0) v = atomicAdd(a.queue, 1u);
        const int64_t wi = (int64_t)__shfl(v, 0, 64);
        if (wi >= n_wave_items) break;
        fit_wave<MODE, CHI2, G>(a, wi, st);
      }
    }
  } else {
    // (with a work order, longest first, blocks keep the hardware order:
    // consecutive items, of similar length, go to different XCDs, where the
    // remap would put the longest eighth of the work on one of them)
    const int nb = gridDim.x, b = blockIdx.x;
    const int per = nb / 8, rem = nb % 8, xcd = b % 8, idx = b / 8;
    const int lb = a.order ? b
                   : (xcd < rem) ? xcd * (per + 1) + idx
                                 : rem * (per + 1) + (xcd - rem) * per + idx;
    const int64_t wi = (int64_t)lb * (blockDim.x >> 6) + (threadIdx.x >> 6);
    fit_wave<MODE, CHI2, G>(a, wi, st);
  }
  if (a.stats) {
    put_stats<MODE>(a.stats, st, lane);
  }
}

// ---------------------------------------------------------------- single epochs

// Sweeps of the simultaneous iteration before a pair's images are tried, and
// passes of that try (see magnify_pairs_kernel).
#define SBLM_PAIR_SWEEPS 1
#define SBLM_PAIR_PASSES 6

// A pair (individual, epoch) p = ind n_t + k: the source, the lens.
__device__ __forceinline__ void pair_setup(const double* theta, const double* t, int64_t n_ind,
                                           int64_t n_t, int64_t p, cx<double>& zeta, double& d,
                                           double& q) {
  const int64_t ind = n_t == 1 ? p : p / n_t;
  const ItemTrig tr = item_trig(theta[ind], theta[3 * n_ind + ind], theta[4 * n_ind + ind]);
  q = tr.q;
  d = theta[n_ind + ind];
  zeta = source_position(t[p - ind * n_t], theta[5 * n_ind + ind], tr.itE, tr.sa, tr.ca,
                         theta[2 * n_ind + ind]);
}

// The cold solve of up to 64 pairs, one per lane, with the output.
template <int MODE>
__device__ __noinline__ void solve_pairs(const double* theta, const double* t, int64_t n_ind,
                                         int64_t n_t, int64_t p, int active, double* A,
                                         int8_t* n_img, LaneStats* cnt) {
  cx<double> zeta;
  double io[11], d, q;
  pair_setup(theta, t, n_ind, n_t, p, zeta, d, q);
  const int out =
      solve_epoch<MODE>(zeta.re, zeta.im, d, q, active ? SOLVE_ACTIVE : 0, io, cnt);
  if (active) {
    A[p] = io[10];
    if (n_img) n_img[p] = (int8_t)(out >> 4);
  }
}

// Magnifications of pairs that share no chain, `batches` times 64 of them per
// wave; blocks of 256 threads.
//   Bound by FP64 arithmetic in lockstep: a cold solve takes 2.7 sweeps, the
// slowest of 64 lanes 7.6.  So a pair gets one sweep, and its three roots of
// least residual go through the checks of a tracked epoch (track_images): over
// the prior 6% fail, and are put aside until they fill a wave of their own.
// (After two sweeps 3% fail, after four 0.4%, but of 64 lanes one in 85% and
// 25% of the cases.)  At the end the block's waves share out what is left; one
// residency of long-lived blocks, so that this, some 15 us of latency, comes
// once: 2^20 single epochs 200 us in lockstep, 147 so (205, 187 and 162 us with
// 2, 3 and 4 batches a wave instead of 8); two sweeps and 3 passes 148 us, one
// and 4 162, one and 8 152.
template <int MODE>
__global__ __launch_bounds__(256, 2) void magnify_pairs_kernel(FitArgs a, int batches) {
  // pairs of each wave still to be solved, and how many at the end
  __shared__ int left[4][128], n_end[4];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t n = a.n_ind * a.n_t;
  const int64_t p0 = ((int64_t)blockIdx.x * 4 + w) * batches * 64;
  int n_left = 0;
  unsigned int tracked = 0, tried = 0;
  WaveStats slow = {};
  for (int b = 0; b < batches && p0 + b * 64 < n; ++b) {
    const int64_t p = p0 + b * 64 + lane;
    const bool active = p < n;
    cx<double> zeta, c[6], z[5];
    double d, q;
    pair_setup(a.theta, a.t, a.n_ind, a.n_t, active ? p : n - 1, zeta, d, q);
    lens_coeffs(zeta, d, q, c);
    cx<float> zf[5];
    bool ok = active && q <= 2.0 && light_secondary_start(zeta, d, q, zf);
    double A = 0.0;
    int nimg = 3;
    if (ok) {
      ++tried;
#pragma unroll
      for (int i = 0; i < 5; ++i) z[i] = {(double)zf[i].re, (double)zf[i].im};
#pragma unroll 1
      for (int k = 0; k < SBLM_PAIR_SWEEPS; ++k)
        (void)aberth_sweep<false>(c, z, false, SBLM_ROOT_TAU, (double*)nullptr);
      // the three roots of least residual
      double r2[5];
#pragma unroll
      for (int i = 0; i < 5; ++i) r2[i] = lens_residual2(z[i], zeta, d, q);
      cx<double> zt[3] = {z[0], z[1], z[2]}, vt[3];
#pragma unroll
      for (int i = 0; i < 5; ++i) {
        int rank = 0;
#pragma unroll
        for (int j = 0; j < 5; ++j)
          rank += (r2[j] < r2[i] || (r2[j] == r2[i] && j < i)) ? 1 : 0;
#pragma unroll
        for (int k = 0; k < 3; ++k)
          if (rank == k) zt[k] = z[i];
      }
      ok = track_images(zt, vt, zeta, {0.0, 0.0}, d, q, A, nimg, SBLM_PAIR_PASSES);
      tracked += ok ? 1u : 0u;
    }
    if (ok) {
      a.A[p] = A;
      if (a.n_img) a.n_img[p] = (int8_t)nimg;
    }
    // those left, in order; solved as soon as they fill a wave (by other lanes:
    // a fence between their reads and the writes on either side)
    const unsigned long long m = __ballot(active && !ok);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (active && !ok)
      left[w][n_left + __popcll(m & ((1ull << lane) - 1ull))] = b * 64 + lane;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    n_left += __popcll(m);
    if (n_left >= 64) {
      n_left -= 64;
      solve_pairs<MODE>(a.theta, a.t, a.n_ind, a.n_t, p0 + left[w][n_left + lane], 1, a.A,
                        a.n_img, &slow);
    }
  }
  // the rest of the block's, shared out anew
  if (lane == 0) n_end[w] = n_left;
  __syncthreads();
  int j = 0, i = w * 64 + lane;
  while (j < 4 && i >= n_end[j]) i -= n_end[j++];
  if (__any(j < 4)) {
    const int64_t p =
        j < 4 ? ((int64_t)blockIdx.x * 4 + j) * batches * 64 + left[j][i] : n - 1;
    solve_pairs<MODE>(a.theta, a.t, a.n_ind, a.n_t, p, j < 4 ? 1 : 0, a.A, a.n_img, &slow);
  }
  if (a.stats) {
    slow.solves += tracked;
    slow.newton += tracked;
    slow.tracked = tracked;
    slow.iters += tried * SBLM_PAIR_SWEEPS;
    slow.wave_iters += tried * SBLM_PAIR_SWEEPS;
    put_stats<MODE>(a.stats, slow, lane);
  }
}

// The kernels are compiled for blocks of at most this many threads.
#define SBLM_FIT_MAX_THREADS 256

template <int MODE, bool CHI2, int G>
static hipError_t launch_gg(const FitArgs& a, hipStream_t s, int wpb) {
  if (wpb < 1 || 64 * wpb > SBLM_FIT_MAX_THREADS) return hipErrorInvalidConfiguration;
  if constexpr (G > 64) {
    // several waves per individual: one-shot grid, lockstep; for chi^2, where
    // they meet at the merge, whole individuals in every block
    const int P = (G == WIDE ? a.lanes_per_ind : G) / 64;
    if (a.queue || (CHI2 && wpb % P != 0)) return hipErrorInvalidConfiguration;
    const size_t smem = ROOT_HIST_BYTES * 64 * wpb + 6 * sizeof(double) * wpb;
    const int64_t nblk = (a.n_ind * P + wpb - 1) / wpb;
    if (nblk <= 0) return hipSuccess;
    hipLaunchKernelGGL((fitness_kernel<MODE, CHI2, G, 0>), dim3((unsigned)nblk),
                       dim3(64 * wpb), smem, s, a);
    return hipGetLastError();
  } else {
    const size_t smem = ROOT_HIST_BYTES * 64 * wpb;
    const int64_t groups_per_block = (int64_t)wpb * (64 / G);
    int64_t nblk = (a.n_ind + groups_per_block - 1) / groups_per_block;
    if (nblk <= 0) return hipSuccess;
    if (!CHI2 && a.queue) return hipErrorInvalidConfiguration;
    constexpr int PF = CHI2 ? 1 : 0;  // (magnifications: the one-shot grid only)
    auto kern = a.queue ? fitness_kernel<MODE, CHI2, G, PF> : fitness_kernel<MODE, CHI2, G, 0>;
    if (a.queue) {  // persistent grid: as many blocks as can be resident
      int dev = 0, ncu = 0, per_cu = 0;
      hipError_t e = hipGetDevice(&dev);
      if (e == hipSuccess) e = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
      if (e == hipSuccess)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, 64 * wpb, smem);
      if (e != hipSuccess) return e;
      const int64_t resident = (int64_t)(per_cu > 0 ? per_cu : 1) * ncu;
      nblk = nblk < resident ? nblk : resident;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)nblk), dim3(64 * wpb), smem, s, a);
    return hipGetLastError();
  }
}

template <int MODE>
static hipError_t launch_pairs(const FitArgs& a, hipStream_t s) {
  const int64_t n = a.n_ind * a.n_t;
  // as many blocks as the chip holds at once, each wave with as many pairs
  const int64_t batches = (n + RESIDENT_LANES - 1) / RESIDENT_LANES;
  if (batches > (1 << 24)) return hipErrorInvalidConfiguration;
  const int64_t nblk = (n + batches * 256 - 1) / (batches * 256);
  hipLaunchKernelGGL((magnify_pairs_kernel<MODE>), dim3((unsigned)nblk), dim3(256), 0, s, a,
                     (int)batches);
  return hipGetLastError();
}

template <int MODE, bool CHI2>
static hipError_t launch_g(const FitArgs& a, hipStream_t s, int wpb) {
  if constexpr (CHI2) {
    if (a.lanes_per_ind == 256) return launch_gg<MODE, CHI2, 256>(a, s, wpb);
    if (a.lanes_per_ind == 128) return launch_gg<MODE, CHI2, 128>(a, s, wpb);
  } else {
    if (a.lanes_per_ind == MAGNIFY_PAIRS) return launch_pairs<MODE>(a, s);
    if (a.lanes_per_ind > 64 && a.lanes_per_ind % 64 == 0)
      return launch_gg<MODE, CHI2, WIDE>(a, s, wpb);
  }
  if (a.lanes_per_ind == 64) return launch_gg<MODE, CHI2, 64>(a, s, wpb);
  if (a.lanes_per_ind == 32) return launch_gg<MODE, CHI2, 32>(a, s, wpb);
  if (a.lanes_per_ind == 8) return launch_gg<MODE, CHI2, 8>(a, s, wpb);
  if constexpr (!CHI2) {
    if (a.lanes_per_ind == 4) return launch_gg<MODE, CHI2, 4>(a, s, wpb);
    if (a.lanes_per_ind == 2) return launch_gg<MODE, CHI2, 2>(a, s, wpb);
    if (a.lanes_per_ind == 1) return launch_gg<MODE, CHI2, 1>(a, s, wpb);
  }
  return launch_gg<MODE, CHI2, 16>(a, s, wpb);
}

hipError_t launch_fitness(const FitArgs& a, int mode, bool chi2,
                          hipStream_t s, int wpb) {
  if (mode == SBLM_MIXED)
    return chi2 ? launch_g<SBLM_MIXED, true>(a, s, wpb)
                : launch_g<SBLM_MIXED, false>(a, s, wpb);
  return chi2 ? launch_g<SBLM_FP64, true>(a, s, wpb)
              : launch_g<SBLM_FP64, false>(a, s, wpb);
}

}  // namespace sblm
