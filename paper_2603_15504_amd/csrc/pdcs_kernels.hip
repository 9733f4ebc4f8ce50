// HIP kernels of the PDCS LP solver for gfx950.
//
// One trial of AdaptiveStepPDHG (Function 2) is three passes and two finalizers:
//   primal   : deferred reflected-Halpern commit of x and of G^T y (Algorithm 1:
//              reflection and averaging), then x_hat = Proj_[l,u](x - tau (c - G^T y))   (eq. PDHG)
//   dual     : SpMV G x_hat and the dual step:
//              Halpern commit of y and of G x, then
//              y_hat = Proj_Kd(y + sigma (h - 2 G x_hat + G x))          (eq. PDHG)
//   fin_ls   : step-size test of Function 2 (eta_bar, eta')
//   lam      : transposed SpMV G^T y_hat with the dual-slack epilogue
//              lam = c - G^T y_hat and its error terms (eq. tolerance-3)
//   fin_beta : reflection parameter (eq. adaptive_reflection)
// Where an instance has few records, fin_ls runs inside the lam pass and fin_beta inside
// the next trial's primal pass, by every workgroup (k_lam_fold, k_band_lam_fold,
// k_lam_epi_fold, k_primal_fold): three launches on row blocks (the dual step ends
// k_dual's rows), four on band tiles of one window (k_band_spmv and k_dual_epi), five
// on several.  Else the finalizers are launches of their own (k_fin_ls, k_fin_beta).
// Instances that fit in LDS run whole chunks of trials in one workgroup (k_trials_lds).
// G x and G^T y of the Halpern iterate are maintained by the same linear
// combination as the iterate, so a trial reads the matrix once (G x_hat) and
// an accepted trial twice (plus G^T y_hat); k_lam_fold and the product on several
// windows read it twice for a rejected trial as well.
//
// Every K trials a restart check runs (Section 2.3): candidate products with
// FP64 values, N-norm radii, the bisection of Algorithm 3 as a multisection
// (kProbes values of t per pass over the vectors), the restart conditions,
// the primal-weight update (Section 2.5) and the termination test (Section 3).
#include "pdcs_dev.h"
#include "pdcs_launch.h"

#include <math.h>

#include <algorithm>
#include <type_traits>

namespace pdcs {

// ===========================================================================
// Second-order-cone row blocks (socG option of Section 3, rescaled cones of
// Section 2.6)
// ===========================================================================
// Projection of one block v (element i read by ld(i)) onto diag(e) K_soc,
// K_soc = {(t, w): ||w|| <= t}, e_i = ef(i) > 0, by one wave; element i of the
// result goes to st(i, p_i), each by the lane that read v_i.  From the KKT
// conditions: v itself inside the cone; 0 inside the polar cone -diag(1/e)
// K_soc (||w e_w|| <= -t e_t); otherwise the multiplier mu > 0 is the root of
//   F(mu) = sum_i v_i^2 e_i^2 / (e_i^2 s + mu)^2 = 1,  s = v_0 / e_0 + mu / e_0^2
// (sum over i >= 1), F decreasing, F > 1 at max(0, -v_0 e_0) and F <= 1 at
// ||w e_w||: Newton steps on 1 - F^-1/2 (linear in mu when one term
// dominates), kept inside the bracket, then p_0 = e_0 s and
// p_i = v_i e_i^2 s / (e_i^2 s + mu).  FP64 throughout; the
// first kSocCache elements of each lane stay in registers.
constexpr int kSocCache = 4;

template <class LD, class EF, class ST>
__device__ __forceinline__ void wave_proj_soc(int d, const LD& ld, const EF& ef, const ST& st) {
  const int lane = threadIdx.x & (kWave - 1);
  const double v0 = ld(0), e0 = ef(0);
  double vr[kSocCache], er[kSocCache];
#pragma unroll
  for (int k = 0; k < kSocCache; ++k) {
    const int i = lane + k * kWave;
    vr[k] = i < d ? ld(i) : 0.0;
    er[k] = i < d ? ef(i) : 1.0;
  }
  // fn(i, v_i, e_i) over this lane's elements i >= 1
  const auto each = [&](auto&& fn) {
#pragma unroll
    for (int k = 0; k < kSocCache; ++k) {
      const int i = lane + k * kWave;
      if (i >= 1 && i < d) fn(i, vr[k], er[k]);
    }
    for (int i = lane + kSocCache * kWave; i < d; i += kWave) fn(i, ld(i), ef(i));
  };
  double in_w = 0.0, po_w = 0.0;
  each([&](int, double v, double e) {
    in_w += (v / e) * (v / e);
    po_w += (v * e) * (v * e);
  });
  in_w = wave_sum(in_w);
  po_w = wave_sum(po_w);
  if (sqrt(in_w) <= v0 / e0) {
    if (lane == 0) st(0, v0);
    each([&](int i, double v, double) { st(i, v); });
    return;
  }
  if (sqrt(po_w) <= -v0 * e0) {
    if (lane == 0) st(0, 0.0);
    each([&](int i, double, double) { st(i, 0.0); });
    return;
  }
  const double ie02 = 1.0 / (e0 * e0);
  double lo = fmax(0.0, -v0 * e0), hi = fmax(lo, sqrt(po_w));
  // phi = 1 - F^-1/2 is < 0 at lo and >= 0 at hi; a Newton step that leaves
  // the bracket is replaced by the secant step of phi over it (bisection while
  // phi is unknown at an end), and one that lands within rounding of an end
  // (the root sits at that end) ends the search there
  double mu = lo, flo = NAN, fhi = NAN;
#pragma unroll 1
  for (int it = 0; it < 200; ++it) {
    const double sv = v0 / e0 + mu * ie02;
    double F = 0.0, dF = 0.0;
    each([&](int, double v, double e) {
      const double e2 = e * e;
      const double den = e2 * sv + mu, q = v * v * e2;
      if (q > 0.0) {  // (a zero term stays zero at den = 0, which mu = 0 with v_0 = 0 gives)
        F += q / (den * den);
        dF -= 2.0 * q * (e2 * ie02 + 1.0) / (den * den * den);
      }
    });
    F = wave_sum(F);
    dF = wave_sum(dF);
    const double rs = 1.0 / sqrt(F);
    const double phi = 1.0 - rs;
    if (F > 1.0) lo = mu, flo = phi;
    else hi = mu, fhi = phi;
    if (F == 1.0 || !(hi > lo) || hi - lo <= 4e-16 * hi) break;
    double next = mu - 2.0 * phi / (rs * rs * rs * dF);
    if (!(next > lo && next < hi)) {
      if (fabs(next - lo) <= 4e-16 * lo) {
        mu = lo;
        break;
      }
      if (fabs(next - hi) <= 4e-16 * hi) {
        mu = hi;
        break;
      }
      next = (flo == flo && fhi == fhi) ? lo - flo * (hi - lo) / (fhi - flo) : 0.5 * (lo + hi);
      if (!(next > lo && next < hi)) next = 0.5 * (lo + hi);
    }
    if (fabs(next - mu) <= 4e-16 * next) {
      mu = next;
      break;
    }
    mu = next;
  }
  const double sv = v0 / e0 + mu * ie02;
  if (lane == 0) st(0, e0 * sv);
  each([&](int i, double v, double e) {
    const double e2 = e * e;
    st(i, v * e2 * sv / (e2 * sv + mu));
  });
}

// ===========================================================================
// Exponential-cone row blocks (expG and dual_expG options of Section 3)
// ===========================================================================
// K_exp = closure {(x, y, z): y > 0, y e^(x / y) <= z}; its dual cone
// K_exp* = closure {(u, v, w): u < 0, -u e^(v / u) <= e w}.
__device__ __forceinline__ bool exp_cone_has(double x, double y, double z) {
  if (y > 0.0) return z > 0.0 && x <= y * log(z / y);
  return y == 0.0 && x <= 0.0 && z >= 0.0;
}

__device__ __forceinline__ bool exp_dual_has(double u, double v, double w) {
  if (u < 0.0) return w > 0.0 && log(-u) + v / u <= 1.0 + log(w);
  return u == 0.0 && v >= 0.0 && w >= 0.0;
}

// (u, v, w) in K_exp* up to 1e-15 of its size (rounding).
__device__ __forceinline__ bool exp_dual_near(double u, double v, double w) {
  const double sc = 1e-15 * (fabs(u) + fabs(v) + fabs(w));
  if (u < -sc) return -u * exp(v / u) <= M_E * w + sc;
  return v >= -sc && w >= -sc;
}

// A point to project onto F K_exp: v, f and 1 / f.
struct ExpPoint {
  double v[3], f[3], fi[3];
};

// Sign of the slope of the angle between v and the boundary ray of F K_exp
// through F a(r), a(r) = (r, 1, e^r): the triple product
// det[v, F a(r), F^-1 n(r)], n(r) = (-1, r - 1, e^-r) the element of K_exp*
// normal to the cone along the ray (F a(r) x F^-1 n(r) points along the
// derivative of the unit ray), times e^r, divided by e^2r for r > 0 so that
// it stays finite.  E = e^r and iE = e^-r are passed in.
__device__ __forceinline__ double exp_ray_turn(double r, double E, double iE, const ExpPoint& P) {
  double a0, a1, a2, m0, m1, m2;  // a = F a(r), m = e^r F^-1 n(r), both times e^-r when r > 0
  if (r <= 0.0) {
    a0 = P.f[0] * r, a1 = P.f[1], a2 = P.f[2] * E;
    m0 = -E * P.fi[0], m1 = E * (r - 1.0) * P.fi[1], m2 = P.fi[2];
  } else {
    a0 = P.f[0] * r * iE, a1 = P.f[1] * iE, a2 = P.f[2];
    m0 = -P.fi[0], m1 = (r - 1.0) * P.fi[1], m2 = iE * P.fi[2];
  }
  return P.v[0] * (a1 * m2 - a2 * m1) + P.v[1] * (a2 * m0 - a0 * m2) + P.v[2] * (a0 * m1 - a1 * m0);
}

// The slope t at r (one exp), its derivative dt and the size sc of the terms
// summed into t (|t| <= 1e-15 sc is rounding noise: r is a root).
__device__ __forceinline__ void exp_ray_turn_d(double r, const ExpPoint& P, double& t, double& dt, double& sc) {
  double a0, a1, a2, m0, m1, m2, da0, da1, da2, dm0, dm1, dm2;
  const double q = exp(-fabs(r));  // e^r for r <= 0, e^-r above
  if (r <= 0.0) {
    const double E = q;
    a0 = P.f[0] * r, a1 = P.f[1], a2 = P.f[2] * E;
    m0 = -E * P.fi[0], m1 = E * (r - 1.0) * P.fi[1], m2 = P.fi[2];
    da0 = P.f[0], da1 = 0.0, da2 = a2;
    dm0 = m0, dm1 = E * r * P.fi[1], dm2 = 0.0;
  } else {  // both vectors times e^-r: the derivative of t e^-2r, whose sign change is the same
    const double iE = q;
    a0 = P.f[0] * r * iE, a1 = P.f[1] * iE, a2 = P.f[2];
    m0 = -P.fi[0], m1 = (r - 1.0) * P.fi[1], m2 = iE * P.fi[2];
    da0 = P.f[0] * (1.0 - r) * iE, da1 = -a1, da2 = 0.0;
    dm0 = 0.0, dm1 = P.fi[1], dm2 = -m2;
  }
  const double c0 = a1 * m2 - a2 * m1, c1 = a2 * m0 - a0 * m2, c2 = a0 * m1 - a1 * m0;
  t = P.v[0] * c0 + P.v[1] * c1 + P.v[2] * c2;
  sc = fabs(P.v[0]) * (fabs(a1 * m2) + fabs(a2 * m1)) + fabs(P.v[1]) * (fabs(a2 * m0) + fabs(a0 * m2)) +
       fabs(P.v[2]) * (fabs(a0 * m1) + fabs(a1 * m0));
  dt = P.v[0] * (da1 * m2 - da2 * m1 + a1 * dm2 - a2 * dm1) + P.v[1] * (da2 * m0 - da0 * m2 + a2 * dm0 - a0 * dm2) +
       P.v[2] * (da0 * m1 - da1 * m0 + a0 * dm1 - a1 * dm0);
}

// Candidate on the ray of r: the nearest point s F a(r), s = <F a, v> / |F a|^2,
// kept in (bd, b) when s > 0 and it is nearer than bd; cert is set when it is
// nearer and v - p is a nonpositive multiple of F^-1 n(r) (at a root of the
// slope v - p is parallel to it): then -F (v - p) lies in K_exp*, p in F K_exp
// and <p, v - p> = 0, which makes p the projection.
__device__ __forceinline__ void exp_ray_candidate(double r, const ExpPoint& P, double& bd, double& b0, double& b1,
                                                  double& b2, bool& cert) {
  const double q = exp(-fabs(r));  // e^r for r <= 0, e^-r above
  const double E = r <= 0.0 ? q : 1.0 / q;
  const double q0 = P.f[0] * r, q1 = P.f[1], q2 = P.f[2] * E;
  const double s = (q0 * P.v[0] + q1 * P.v[1] + q2 * P.v[2]) / (q0 * q0 + q1 * q1 + q2 * q2);
  if (!(s > 0.0)) return;
  const double c0 = s * q0, c1 = s * q1, c2 = s * q2;
  const double d0 = P.v[0] - c0, d1 = P.v[1] - c1, d2 = P.v[2] - c2;
  const double d = d0 * d0 + d1 * d1 + d2 * d2;
  // m = F^-1 n(r) min(1, e^r); at a root v - p is parallel to m, so the cosine
  // of their angle is -1 (the projection) or +1 (not): the test takes the
  // sign with room for rounding, and a residual at the rounding level of v
  // (v on the boundary: p is then within that level of the projection)
  const double m0 = r <= 0.0 ? -E * P.fi[0] : -P.fi[0];
  const double m1 = r <= 0.0 ? (r - 1.0) * E * P.fi[1] : (r - 1.0) * P.fi[1];
  const double m2 = r <= 0.0 ? P.fi[2] : q * P.fi[2];
  const double w = d0 * m0 + d1 * m1 + d2 * m2;
  const double vv = P.v[0] * P.v[0] + P.v[1] * P.v[1] + P.v[2] * P.v[2];
  const bool ok = w <= 0.5 * sqrt(d * (m0 * m0 + m1 * m1 + m2 * m2)) || d <= 1e-24 * vv;
  // a certified candidate is the projection: it replaces an uncertified one
  // even when rounding makes it look no nearer (near the apex the face clip
  // and the projection can be within rounding of the same distance from v
  // while the points differ by the square root of that rounding)
  if (!((ok && !cert) || (ok == cert && d < bd))) return;
  bd = d, b0 = c0, b1 = c1, b2 = c2, cert = ok;
}

// One scan of the rays by the wave: lane l takes cells [l C, l C + C) of
// width h from r = -32 C h, every + to - sign change of the slope is refined
// to full precision and its candidate kept (exp_ray_candidate).  e^r runs by
// multiplication with g = e^h (ig = e^-h) along a lane's cells (the
// refinement uses exp itself).
// (Loops are kept rolled throughout, so that each kernel holds one compact
// copy of the projection.)
__device__ __forceinline__ void exp_scan(int C, double h, double g, double ig, const ExpPoint& P, double& bd,
                                         double& b0, double& b1, double& b2, bool& cert) {
  const int lane = threadIdx.x & (kWave - 1);
  const double r_first = -0.5 * kWave * C * h;
  int k = lane * C;
  double lo = r_first + k * h;
  const double q = exp(-fabs(lo));
  double E = lo <= 0.0 ? q : 1.0 / q, iE = lo <= 0.0 ? 1.0 / q : q;
  double t_lo = exp_ray_turn(lo, E, iE, P);
#pragma unroll 1
  for (int c = 0; c < C; ++c) {
    ++k;
    const double hi = r_first + k * h;
    E *= g, iE *= ig;
    const double t_hi = exp_ray_turn(hi, E, iE, P);
    if (t_lo > 0.0 && t_hi <= 0.0) {
      // Newton steps from the secant point of the cell, kept inside the
      // bracket [x, z] (slope > 0 at x, <= 0 at z; bisection when a step
      // leaves it), until the slope is rounding noise
      double x = lo, z = hi;
      double r = (lo * t_hi - hi * t_lo) / (t_hi - t_lo);
      if (!(r > x && r < z)) r = 0.5 * (x + z);
#pragma unroll 1
      for (int it = 0; it < 100; ++it) {
        double t, dt, sc;
        exp_ray_turn_d(r, P, t, dt, sc);
        if (fabs(t) <= 1e-15 * sc) break;
        if (t > 0.0) x = r;
        else z = r;
        double nr = r - t / dt;
        if (!(nr > x && nr < z)) nr = 0.5 * (x + z);
        if (!(nr > x && nr < z)) break;
        r = nr;
      }
      exp_ray_candidate(r, P, bd, b0, b1, b2, cert);
    }
    lo = hi;
    t_lo = t_hi;
  }
}

// Best candidate over the wave: certified before uncertified, then the nearest
// (ties: the lowest lane), among the lanes that hold a certified candidate or,
// when need_cert is false, among all.  Returns whether any lane took part.
__device__ __forceinline__ bool exp_wave_pick(double bd, double b0, double b1, double b2, bool cert, bool need_cert,
                                              double (&p)[3]) {
  const int lane = threadIdx.x & (kWave - 1);
  const bool eligible = cert || !need_cert;
  double d = eligible ? bd : INFINITY;
  int who = eligible ? lane : kWave;
  int rank = cert ? 0 : 1;
  for (int off = 1; off < kWave; off <<= 1) {
    const double od = __shfl_xor(d, off);
    const int ow = __shfl_xor(who, off), orank = __shfl_xor(rank, off);
    const double o0 = __shfl_xor(b0, off), o1 = __shfl_xor(b1, off), o2 = __shfl_xor(b2, off);
    if (ow < kWave &&
        (who == kWave || orank < rank || (orank == rank && (od < d || (od == d && ow < who)))))
      d = od, who = ow, rank = orank, b0 = o0, b1 = o1, b2 = o2;
  }
  if (who == kWave) return false;
  p[0] = b0, p[1] = b1, p[2] = b2;
  return true;
}

// The projection among the face's clip and the best points of the rays
// s F a(r), by one wave: the local maxima of the angle along the rays (+ to -
// sign changes of exp_ray_turn) and, for rays below the scanned range, whose
// third coordinate is then below e^-300 of the others, the ray through v's own
// x / y, r = (v_1 / f_1) / (v_2 / f_2).  A first scan on a
// coarse grid (step 0.4 over |r| <= 307.2) ends the search when a candidate
// carries the projection's certificate; else a scan on a fine grid (step
// 0.05 over |r| <= 300.8) takes a certified candidate if one turns up, else
// the nearest of all candidates.  Above the
// scanned range the rays lie within e^-300 of the face's edge (0, 0, 1).
constexpr double kExpTail = -300.0;

__device__ __forceinline__ void exp_scan_wave(const ExpPoint& P, double (&p)[3]) {
  const double face[3] = {fmin(P.v[0], 0.0), 0.0, fmax(P.v[2], 0.0)};
  const double face_d =
      (P.v[0] - face[0]) * (P.v[0] - face[0]) + P.v[1] * P.v[1] + (P.v[2] - face[2]) * (P.v[2] - face[2]);
  const bool tail = P.v[0] < 0.0 && P.v[1] > 0.0 && (P.v[0] * P.fi[0]) / (P.v[1] * P.fi[1]) < kExpTail;
  const int lane = threadIdx.x & (kWave - 1);
#pragma unroll 1
  for (int pass = 0; pass < 2; ++pass) {  // coarse, then fine
    double bd = face_d, b0 = face[0], b1 = face[1], b2 = face[2];
    bool cert = false;
    if (tail && lane == 0) exp_ray_candidate((P.v[0] * P.fi[0]) / (P.v[1] * P.fi[1]), P, bd, b0, b1, b2, cert);
    // e^0.4, e^-0.4, e^0.05, e^-0.05 to double precision
    exp_scan(pass == 0 ? 24 : 188, pass == 0 ? 0.4 : 0.05, pass == 0 ? 1.4918246976412703 : 1.0512710963760241,
             pass == 0 ? 0.6703200460356393 : 0.951229424500714, P, bd, b0, b1, b2, cert);
    if (exp_wave_pick(bd, b0, b1, b2, cert, pass == 0, p)) return;
  }
}

// The projection by one lane; returns whether p is certified.
//
// With w = v / f and z = f v, a point outside the cone, its polar and the
// face's reach projects onto s F a(r), s > 0, with v - p = -t F^-1 n(r), t > 0,
// and r is the one root of the slope in V = {psi < 0, chi > 0}.  At an end of an
// interval of V the slope is positive where r enters it and negative where r
// leaves it, so an interval with both ends holds a root: only one such interval
// can exist, and the side of the root is known for every r outside V too.
//   psi is convex in r for w_2 > 0 and concave for w_2 < 0; for w_1, w_2 > 0 it
//   is lowest, and negative, at log(w_2 / w_1): psi >= 0 is then beyond the root
//   on that seed's right and before it on its left; otherwise psi >= 0 lies
//   beyond the root for w_1 > 0 and before it for w_1 <= 0.
//   chi likewise with -z_2, z_0: highest, and positive, at log(z_0 / -z_2) for
//   z_0 > 0 > z_2; otherwise chi <= 0 lies before the root for z_0 > 0 and
//   beyond it for z_0 <= 0.
// From a seed in the root's neighbourhood: Newton steps of the slope, steps of
// growing length while the root has no bracket, bisection where Newton leaves
// the bracket.  It is bound by its chain of dependent operations: 6 to 8 slopes
// at the median over points of 16 decades and factors of 6, at most 24, 3 us for
// one point and 6 us for 64.  (131072 projections of ordinary points: 20 us, 402 us
// with a wave's scan of 1537 rays for each.)
__device__ __forceinline__ bool exp_lane(const ExpPoint& P, double (&p)[3]) {
  const double w0 = P.v[0] * P.fi[0], w1 = P.v[1] * P.fi[1], w2 = P.v[2] * P.fi[2];
  const double z0 = P.v[0] * P.f[0], z1 = P.v[1] * P.f[1], z2 = P.v[2] * P.f[2];
  double bd = INFINITY;
  bool cert = false;
  if (w0 < 0.0 && w1 > 0.0 && w0 / w1 < kExpTail) {
    exp_ray_candidate(w0 / w1, P, bd, p[0], p[1], p[2], cert);
    return cert;
  }
  const bool low = w1 > 0.0 && w2 > 0.0, high = w2 < 0.0 && w0 > 0.0;
  const bool far = !low && !high && w2 > 0.0 && w1 <= 0.0;  // e^r / r = w_2 / w_0, nearly
  const double lg = log((low || far ? w2 : (high ? -z0 : 1.0)) / (low ? w1 : (far ? w0 : (high ? z2 : 1.0))));
  double seed = lg;
  if (far) seed = fmax(1.0, lg + log(fmax(lg, 1.0)));
  else if (!low && !high) seed = w1 > 0.0 ? (w0 <= 0.0 ? w0 / w1 : 0.5) : fmax(1.0, 1.0 - z1 / z0);
  const double k0 = P.v[0] * P.f[1] * P.fi[2], k1 = P.v[0] * P.f[2] * P.fi[1], k2 = P.v[1] * P.f[2] * P.fi[0];
  const double k3 = P.v[1] * P.f[0] * P.fi[2], k4 = P.v[2] * P.f[0] * P.fi[1], k5 = P.v[2] * P.f[1] * P.fi[0];
  double r = seed, lo = -INFINITY, hi = INFINITY, reach = 2.0, last = INFINITY;
#pragma unroll 1
  for (int it = 0; it < 80; ++it) {
    // slope, its derivative and size as in exp_ray_turn_d, in powers of r with the
    // six products of v, f and 1 / f gathered: half the operations
    const double q = exp(-fabs(r)), r1 = r - 1.0, rr = r * r1;
    const bool neg = r <= 0.0;
    const double x = neg ? q : 1.0, y = neg ? 1.0 : q, x2 = x * x, y2 = y * y;
    const double u = k0 - k3 * r, w = k1 * r1 + k2, g = k4 * rr + k5;
    const double t = u * y2 - w * x2 + q * g;
    const double sc = (fabs(k0) + fabs(k3 * r)) * y2 + (fabs(k1 * r1) + fabs(k2)) * x2 +
                      q * (fabs(k4 * rr) + fabs(k5));
    const double dg = k4 * (r + r1), qg = q * (neg ? dg + g : dg - g);
    const double dt = neg ? qg - k3 - (k1 + 2.0 * w) * x2 : qg - k1 - (k3 + 2.0 * u) * y2;
    const double psi = (w1 * r1 - w0) * x + w2 * y, chi = (z0 * r + z1) * y + z2 * x;
    const bool in = psi < 0.0 && chi > 0.0;
    if (in && fabs(t) <= 1e-15 * sc) break;
    const bool beyond =
        in ? t <= 0.0 : (psi >= 0.0 ? (low ? r > seed : w1 > 0.0) : (high ? r > seed : w0 <= 0.0));
    if (beyond) hi = r;
    else lo = r;
    const bool both = lo > -INFINITY && hi < INFINITY;
    const double inv = __builtin_amdgcn_rcp(dt);  // one refinement: the step needs no more
    const double step = -t * (inv * (2.0 - dt * inv));
    double next = r + step;
    const bool newton = in && dt < 0.0;
    if (newton && fabs(step) <= 0x1p-52 * fabs(r)) break;  // no ray between this one and the root
    if (!(newton && next > lo && next < hi && (both || fabs(step) <= reach)) ||
        (both && it >= 8 && fabs(step) > 0.5 * last))  // (a Newton step that does not shrink: a cycle)
      next = both ? 0.5 * (lo + hi) : (beyond ? r - reach : r + reach);
    if (!(next > lo && next < hi)) break;
    if (!both) reach *= 4.0;
    last = fabs(next - r);
    r = next;
  }
  exp_ray_candidate(r, P, bd, p[0], p[1], p[2], cert);
  return cert;
}

// Projection of v onto F K_exp, F = diag(f) > 0, of each active lane's own point; all
// lanes of the wave call it together.  v itself if v / f is in K_exp; 0 if -F v is in
// K_exp* (the polar cone); the clip onto the face {(x, 0, z): x <= 0, z >= 0} if -F times
// its residual is in K_exp* up to rounding (then the clip is within rounding
// of the projection: this takes the points whose projection lies on a ray
// so far out that it meets the face's edge to working precision); otherwise
// the point of the ray at the root of the slope that carries the projection's
// certificate (exp_lane), and where a lane finds none, the wave's scan for that
// lane (exp_scan_wave), one lane after the other: none of 6e6 points of 16 decades
// and factors of 12, on the cone's boundary, near the apex or in the coordinate planes
// took it, only points whose squares leave FP64's range.
__device__ __forceinline__ void exp_proj_lanes(bool active, const double (&v)[3], const double (&f)[3],
                                               double (&p)[3]) {
  bool done = true;
  if (active) {
    ExpPoint P;
    for (int i = 0; i < 3; ++i) P.v[i] = v[i], P.f[i] = f[i], P.fi[i] = 1.0 / f[i];
    const double c0 = fmin(v[0], 0.0), c2 = fmax(v[2], 0.0);
    if (exp_cone_has(v[0] / f[0], v[1] / f[1], v[2] / f[2])) {
      p[0] = v[0], p[1] = v[1], p[2] = v[2];
    } else if (exp_dual_has(-f[0] * v[0], -f[1] * v[1], -f[2] * v[2])) {
      p[0] = p[1] = p[2] = 0.0;
    } else if (exp_dual_near(-f[0] * (v[0] - c0), -f[1] * v[1], -f[2] * (v[2] - c2))) {
      p[0] = c0, p[1] = 0.0, p[2] = c2;
    } else {
      done = exp_lane(P, p);
    }
  }
  const int lane = threadIdx.x & (kWave - 1);
#pragma unroll 1
  for (unsigned long long left = __ballot(!done); left; left &= left - 1) {
    const int from = __ffsll(left) - 1;
    ExpPoint P;
    for (int i = 0; i < 3; ++i) {
      P.v[i] = __shfl(v[i], from);
      P.f[i] = __shfl(f[i], from);
      P.fi[i] = 1.0 / P.f[i];
    }
    double q[3];
    exp_scan_wave(P, q);
    if (lane == from) p[0] = q[0], p[1] = q[1], p[2] = q[2];
  }
}

// Projection of a 3-row block per active lane onto F K_exp (dual = false) or onto
// F K_exp* (dual = true: F K_exp* is the dual cone of F^-1 K_exp, so by Moreau's
// decomposition P(v) = v + P_{F^-1 K_exp}(-v)); ld, ef and st as in
// wave_proj_soc, called by the block's lane for its three elements.
template <class LD, class EF, class ST>
__device__ __forceinline__ void lanes_proj_exp(bool active, bool dual, const LD& ld, const EF& ef, const ST& st) {
  double v[3] = {0.0, 0.0, 0.0}, f[3] = {1.0, 1.0, 1.0}, w[3], g[3], q[3] = {0.0, 0.0, 0.0};
  if (active)
    for (int i = 0; i < 3; ++i) v[i] = ld(i), f[i] = ef(i);
  for (int i = 0; i < 3; ++i) {
    w[i] = dual ? -v[i] : v[i];
    g[i] = dual ? 1.0 / f[i] : f[i];
  }
  exp_proj_lanes(active, w, g, q);
  if (active)
    for (int i = 0; i < 3; ++i) st(i, dual ? v[i] + q[i] : q[i]);
}

// Cone block kinds of the block table.
constexpr int kConeSoc = 0, kConeExp = 1, kConeDualExp = 2;

// Who handles a cone block: a wave (second-order cones) or one lane of a wave
// whose other lanes have blocks of their own or none (exponential cones).
// any(c) restricts the task to c and says whether the wave has work left;
// elements of the block: for (i = first(); i < count(dim); i += stride()).
struct WaveTask {
  __device__ __forceinline__ bool any(bool c) const { return c; }
  __device__ __forceinline__ int first() const { return threadIdx.x & (kWave - 1); }
  __device__ __forceinline__ int count(int dim) const { return dim; }
  __device__ __forceinline__ int stride() const { return kWave; }
};
struct LaneTask {
  bool active;
  __device__ __forceinline__ bool any(bool c) {
    active = active && c;
    return true;
  }
  __device__ __forceinline__ int first() const { return 0; }
  __device__ __forceinline__ int count(int dim) const { return active ? dim : 0; }
  __device__ __forceinline__ int stride() const { return 1; }
};

// Projection of one cone block of kind `kind` at a primal site (the cone of
// G x - h: K_soc, K_exp or K_exp*) or a dual site (the cone of y, its dual:
// K_soc, K_exp* or K_exp), rescaled by diag(ef).
template <class LD, class EF, class ST>
__device__ __forceinline__ void proj_cone(const WaveTask&, int, bool, int d, const LD& ld, const EF& ef, const ST& st) {
  wave_proj_soc(d, ld, ef, st);
}
template <class LD, class EF, class ST>
__device__ __forceinline__ void proj_cone(const LaneTask& t, int kind, bool dual_site, int, const LD& ld, const EF& ef,
                                          const ST& st) {
  lanes_proj_exp(t.active, (kind == kConeExp) == dual_site, ld, ef, st);
}

// The cone blocks of row range b, each with S independent tasks (sub = 0 ..
// S - 1): fn(who, first row, dimension, kind, sub).  Second-order cones, the first
// in the table, go to the waves: task j of the range (block j / S, sub j mod S) to
// wave j mod kWavesPerBlock.  Exponential cones go to the threads, task j to thread
// j mod kBlock, so that sub is a thread's own where S divides kBlock; a wave takes
// part with all its lanes or none.
// (The dual epilogue of a problem with 310 second-order and 650 exponential cones,
// two tasks each: 18.0 us with a wave for every cone, 12.0 us.)
template <int S, class FN>
__device__ __forceinline__ void for_cone_tasks(const Ranges& R, int b, const FN& fn) {
  static_assert(kBlock % S == 0, "a thread keeps its sub");
  if (!R.blk_soc0) return;
  const int wave = threadIdx.x / kWave;
  const int q0 = R.blk_soc0[b], qe = R.blk_exp0[b], q1 = R.blk_soc1[b];
#pragma unroll 1
  for (int j = wave; j < (qe - q0) * S; j += kWavesPerBlock) {
    const int q = q0 + j / S;
    fn(WaveTask{}, R.soc_r0[q], R.soc_dim[q], kConeSoc, j % S);
  }
#pragma unroll 1
  for (int j0 = wave * kWave; j0 < (q1 - qe) * S; j0 += kBlock) {
    const int j = j0 + (int)(threadIdx.x & (kWave - 1));
    const LaneTask who{j < (q1 - qe) * S};
    const int q = who.active ? qe + j / S : qe;
    fn(who, R.soc_r0[q], 3, (int)R.soc_kind[q], j % S);
  }
}

template <class FN>
__device__ __forceinline__ void for_cone_blocks(const Ranges& R, int b, const FN& fn) {
  for_cone_tasks<1>(R, b, [&](auto who, int r0, int dim, int kind, int) { fn(who, r0, dim, kind); });
}

// Copies of one launch (blockIdx.y), passed by value: the lists need no memory of
// their own that would have to outlive the launch.  (A batch of 128 LPs hands over
// 384 vectors of 60 to 550 doubles: a launch for each and a wait per instance were
// 4.3 ms of its 5.8 ms.)
constexpr int kCopyList = 128;  // 3 KB of the 4 KB of arguments
struct CopyList {
  CopyItem item[kCopyList];
};

__global__ __launch_bounds__(kBlock) void k_copies(CopyList list) {
  const CopyItem c = list.item[blockIdx.y];
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < c.len; i += (int64_t)gridDim.x * kBlock)
    c.dst[i] = c.src[i];
}

// Projection of count vectors of dimension dim (v, f and out: dim doubles
// each, contiguous) onto diag(f) K, K = K_soc (cone 0), K_exp (cone 1) or
// K_exp* (cone 2, dim 3), one wave each (cone 0) or one lane each.
__global__ __launch_bounds__(kBlock) void k_proj_cone(int cone, int dim, const double* __restrict__ v,
                                                      const double* __restrict__ f, double* __restrict__ out,
                                                      int64_t count) {
  const int64_t q = cone == 0 ? (int64_t)blockIdx.x * kWavesPerBlock + threadIdx.x / kWave
                              : (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (cone == 0 && q >= count) return;
  const size_t o = (size_t)q * dim;
  const auto ld = [&](int i) { return v[o + i]; };
  const auto ef = [&](int i) { return f[o + i]; };
  const auto st = [&](int i, double p) { out[o + i] = p; };
  if (cone == 0) wave_proj_soc(dim, ld, ef, st);
  else lanes_proj_exp(q < count, cone == 2, ld, ef, st);
}

// ===========================================================================
// Iteration kernels
// ===========================================================================

// F1: line-search decision of Function 2 for an active instance, from the sums of
// the primal records (p) and the dual records (q); one thread.
// pf: when non-null, pf[0] = (kbar + 1)^-0.3 and pf[1] = (kbar + 1)^-0.6 for the
// kbar this trial reaches, computed beforehand by an otherwise idle thread
__device__ __forceinline__ void fin_ls_apply(Inst& I, const double (&p)[2], const double (&q)[4], const double* pf,
                                             bool traced) {
  I.pending = 0;
  I.check_due = 0;
  I.kbar += 1;
  if (I.precision == kFP64) I.fp64_iters += 1;
  const double dx2 = p[0], dy2 = q[0], dydg = q[1];
  const double omega = I.omega, eta = I.eta;
  const double num = 0.5 * (omega * dx2 + dy2 / omega);
  const double den = fabs(dydg);
  const double etabar = den > 0.0 ? num / den : (double)INFINITY;
  const double kb1 = (double)I.kbar + 1.0;
  const double p3 = pf ? pf[0] : pow(kb1, -0.3), p6 = pf ? pf[1] : pow(kb1, -0.6);
  const double eta_next = fmin((1.0 - p3) * etabar, (1.0 + p6) * eta);
  const bool bad = !isfinite(num) || isnan(etabar) || isnan(q[2]) || isnan(q[3]) || isnan(p[1]) ||
                   !(eta_next > 0.0) || !isfinite(eta_next);
  if (traced && I.trace && I.kbar <= I.trace_cap) {
    double* tr = I.trace + (I.kbar - 1) * kTraceStride;
    tr[0] = (double)I.kbar;
    tr[1] = eta;
    tr[2] = etabar;
    tr[3] = dx2;
    tr[4] = dy2;
    tr[5] = dydg;
    tr[6] = eta < etabar ? 1.0 : 0.0;
    tr[7] = eta_next;
    for (int f = 8; f < kTraceStride; ++f) tr[f] = NAN;
    tr[9] = (double)I.k;
    if (bad) {  // the failing trial's reductions, for diagnosis
      tr[10] = p[1];
      tr[11] = q[3];
      tr[14] = q[2];
    }
  }
  if (bad) {
    I.status = kDone;
    I.exit_code = 8;
    I.last_acc = 0;
    return;
  }
  if (eta < etabar) {
    I.last_acc = 1;
    I.eta_k = eta;
    I.eta_hat = eta_next;
    I.accepted += 1;
    I.dx2 = dx2;
    I.dy2 = dy2;
    I.dydgdx = dydg;
    I.errp2 = q[2];
    I.hy = q[3];
    I.cx = p[1];
  } else {
    I.last_acc = 0;
    if (I.kbar >= I.max_iter) {
      I.status = kDone;
      I.exit_code = 1;
    }
  }
  I.eta = eta_next;
}

// One workgroup per instance.
__device__ __forceinline__ void fin_ls_body(int iid, const int32_t* iblk_p, const double* rec_p,
                                            const int32_t* iblk_d, const double* rec_d, Inst* inst,
                                            const double* pf = nullptr) {
  __shared__ double lds[kWavesPerBlock * 4];
  Inst& I = inst[iid];
  if (I.status != kActive) return;
  double p[2], q[4];
  reduce_records<2, 2>(rec_p, iblk_p[iid], iblk_p[iid + 1], lds, p);
  reduce_records<4, 4>(rec_d, iblk_d[iid], iblk_d[iid + 1], lds, q);
  if (threadIdx.x != 0) return;
  fin_ls_apply(I, p, q, pf, true);
}

// F2: reflection parameter at z_hat (eq. adaptive_reflection with the relative
// errors of eq. tolerance-2), then schedule the Halpern commit.
// For an active instance whose trial was accepted, from the sums of the dual-slack
// records; one thread.
__device__ __forceinline__ void fin_beta_apply(Inst& I, const double (&q)[3], bool traced) {
  const double errp = sqrt(I.errp2), errd = sqrt(q[0]);
  const double pobj = I.cx;
  const double dobj = I.hy + q[1] - q[2];
  const double gap = fabs(pobj - dobj);
  const double rp = errp / (1.0 + I.h1);
  const double rd = errd / (1.0 + I.c1);
  const double rg = gap / (1.0 + fabs(pobj) + fabs(dobj));
  const double me = fmax(rp, fmax(rd, rg));
  if (isnan(me) || isnan(rp) || isnan(rd) || isnan(rg)) {
    I.status = kDone;
    I.exit_code = 8;
    return;
  }
  const double beta = me > 0.0 ? clampd(-0.1 * log10(me) + 0.2, 0.0, 1.0) : 1.0;
  if (traced && I.trace && I.kbar <= I.trace_cap) {
    double* tr = I.trace + (I.kbar - 1) * kTraceStride;
    tr[8] = beta;
    tr[10] = I.cx;
    tr[11] = I.hy;
    tr[12] = q[1];
    tr[13] = q[2];
    tr[14] = I.errp2;
    tr[15] = q[0];
  }
  const double k = (double)I.k;
  I.beta = beta;
  I.ca = (k + 1.0) / (k + 2.0);
  I.cb = 1.0 / (k + 2.0);
  I.pending = 1;
  I.sum_eta += I.eta_k;
  I.k += 1;
  I.check_due = (I.kbar % I.check_every) == 0 ? 1 : 0;
  if (!I.check_due && I.kbar >= I.max_iter) {
    I.status = kDone;
    I.exit_code = 1;
  }
}

// One workgroup per instance.
__device__ __forceinline__ void fin_beta_body(int iid, const int32_t* iblk_l, const double* rec_l, Inst* inst) {
  __shared__ double lds[kWavesPerBlock * 3];
  Inst& I = inst[iid];
  if (I.status != kActive || I.last_acc == 0) return;
  double q[3];
  reduce_records<3, 3>(rec_l, iblk_l[iid], iblk_l[iid + 1], lds, q);
  if (threadIdx.x != 0) return;
  fin_beta_apply(I, q, true);
}

// Finalizers folded into the passes that follow them.  Where an instance has few
// records, every workgroup of the dual-slack pass reduces them and takes the
// line-search decision by itself, and every workgroup of the next primal pass the
// reflection parameter, instead of waiting for a kernel of one workgroup per
// instance; all of them compute the same bits.  The instance record alternates
// between two arrays: the dual-slack pass reads `inst` and its first workgroup of
// an instance writes the record after the decision to `inst2`, the primal pass
// reads `inst2` and its first workgroup writes `inst`, so that no workgroup reads
// what another one of its launch writes.  Ahead of the folded step, the pass has
// requested its own operands.
constexpr int kInstWords = (int)(sizeof(Inst) / 8);
static_assert(sizeof(Inst) % 8 == 0 && kInstWords <= kBlock, "an instance record is copied with one word per thread");

struct FoldIn {  // the instance's records of the two passes before (dual slack: of the one before)
  const int32_t *iblk_a, *iblk_b;
  const double *rec_a, *rec_b;
  const Inst* in;
  Inst* out;
};

// Whether a folded pass has nothing to do for an instance: one that is done, or iterates
// in the other precision (the whole workgroup's answer).  IDLE: there are such instances
// (the host knows when it enqueues a chunk), and every workgroup asks before it requests
// its operands; without any, the operands do not wait for the record (0.4 us a trial of
// m = 2e4, n = 4e4, nnz = 3e5).
// (7 LPs of 4e4 x 8e4, 4.8e5 nonzeros, a trial on row blocks: 81 us with all running, and
// with one running 51 asked after the operands, 27 before, where it takes 26 alone; on
// band tiles 83, 54 and 47.)
template <bool IDLE>
__device__ __forceinline__ bool fold_idle(const FoldIn& f, int iid, int prec) {
  return IDLE && (f.in[iid].status != kActive || f.in[iid].precision != prec);
}

__device__ __forceinline__ void inst_copy_in(Inst* S, const Inst* in) {
  if ((int)threadIdx.x < kInstWords)
    reinterpret_cast<uint64_t*>(S)[threadIdx.x] = reinterpret_cast<const uint64_t*>(in)[threadIdx.x];
}
__device__ __forceinline__ void inst_copy_out(Inst* out, const Inst* S) {
  if ((int)threadIdx.x < kInstWords)
    reinterpret_cast<uint64_t*>(out)[threadIdx.x] = reinterpret_cast<const uint64_t*>(S)[threadIdx.x];
}

// The record of an instance without work here, by the workgroup that writes it.
__device__ __forceinline__ void fold_pass_on(const FoldIn& f, int iid, int prec, bool first) {
  if (first && f.in[iid].precision == prec) inst_copy_out(f.out + iid, f.in + iid);
}

// The line-search decision, in the dual-slack pass.  load() before the pass's own
// loads, decide() (every thread) after them; then S is the instance's record.
struct FoldLds {
  double a[kWavesPerBlock * 2], b[kWavesPerBlock * 4], pf[2];
};
struct FoldLs {
  double p[2], q[4];
  int64_t kbar;
  __device__ __forceinline__ void load(const FoldIn& f, int iid, Inst* S) {
    inst_copy_in(S, f.in + iid);
    records_load<2>(f.rec_a, f.iblk_a[iid], f.iblk_a[iid + 1], p);
    records_load<4>(f.rec_b, f.iblk_b[iid], f.iblk_b[iid + 1], q);
    kbar = f.in[iid].kbar;
  }
  // The waves' sums and, in the workgroup that writes the record, the line-search
  // powers (two lanes of the last wave): work for the time the pass's loads take.
  __device__ __forceinline__ void early(FoldLds& L, bool first) const {
    if (first && threadIdx.x >= kBlock - 2) {
      const int e = kBlock - 1 - (int)threadIdx.x;
      L.pf[e] = pow((double)kbar + 2.0, e ? -0.6 : -0.3);
    }
    records_store<2>(p, L.a);
    records_store<4>(q, L.b);
  }
  __device__ __forceinline__ void decide(const FoldIn& f, FoldLds& L, int iid, Inst* S, int prec, bool first) const {
    __syncthreads();
    if (threadIdx.x == 0 && S->status == kActive && S->precision == prec) {
      double ps[2], qs[4];
      records_total<2>(L.a, ps);
      records_total<4>(L.b, qs);
      // (the others only need to know whether the trial is accepted: any factors in (0, 1) do)
      const double f2[2] = {first ? L.pf[0] : 0.5, first ? L.pf[1] : 0.5};
      fin_ls_apply(*S, ps, qs, f2, first);
    }
    __syncthreads();
    // (in a batch whose instances iterate in both precisions the other one's pass follows:
    // it must not put back the record it read)
    if (first && S->precision == prec) inst_copy_out(f.out + iid, S);
  }
};

// The reflection parameter, in the primal pass of the next trial.
struct FoldBeta {
  double q[3];
  __device__ __forceinline__ void load(const FoldIn& f, int iid, Inst* S) {
    inst_copy_in(S, f.in + iid);
    records_load<3>(f.rec_a, f.iblk_a[iid], f.iblk_a[iid + 1], q);
  }
  __device__ __forceinline__ void decide(const FoldIn& f, int iid, Inst* S, int prec, bool first) {
    __shared__ double lq[kWavesPerBlock * 3];
    records_store<3>(q, lq);
    __syncthreads();
    const bool mine = S->precision == prec;
    if (threadIdx.x == 0 && S->status == kActive && S->last_acc != 0 && mine) {
      double qs[3];
      records_total<3>(lq, qs);
      fin_beta_apply(*S, qs, first);
    }
    __syncthreads();
    if (first && mine) inst_copy_out(f.out + iid, S);
  }
};

// The last reflection parameter of a chunk: from inst2 back to inst.
__global__ __launch_bounds__(kBlock) void k_fold_end(FoldIn f) {
  __shared__ Inst S;
  __shared__ double lq[kWavesPerBlock * 3];
  const int iid = blockIdx.x;
  if (f.out[iid].status != kActive) return;  // its record stayed there
  double q[3];
  inst_copy_in(&S, f.in + iid);
  records_load<3>(f.rec_a, f.iblk_a[iid], f.iblk_a[iid + 1], q);
  records_store<3>(q, lq);
  __syncthreads();
  if (threadIdx.x == 0 && S.status == kActive && S.last_acc != 0) {
    double qs[3];
    records_total<3>(lq, qs);
    fin_beta_apply(S, qs, true);
  }
  __syncthreads();
  inst_copy_out(f.out + iid, &S);
}

// K3: primal step over the columns of the instance.
// The five passes of a trial are device functions of the workgroup's range or
// instance, so that k_trials_wg can run them back to back inside one workgroup.
// They are bound by the latency of their loads: each takes U elements per thread
// at a time and requests all of their operands before the first is used
// (elements past the end repeat the last one and are not stored).
constexpr int kElems = 4;  // elements per thread of the passes over global memory
template <typename T, int U, int NT = kBlock>
struct PrimalElems {
  T x[U], g[U], xh[U], gh[U], xa[U], ga[U], sx[U], c[U], lo[U], hi[U];
  __device__ __forceinline__ void load(const IterPtrs<T>& it, const DataPtrs<T>& d, int j0, int j1, bool commit,
                                       bool avg) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = min(j0 + u * NT, j1 - 1);
      x[u] = it.x[j], g[u] = it.gty[j], c[u] = d.c[j], lo[u] = d.l[j], hi[u] = d.u[j];
      if (commit) xh[u] = it.xh[j], gh[u] = it.gtyh[j], xa[u] = it.xa[j], ga[u] = it.gtya[j];
      if (avg) sx[u] = it.sx[j];
    }
  }
  __device__ __forceinline__ void step(const IterPtrs<T>& it, const Inst& I, int j0, int j1, double (&acc)[2]) const {
    const bool commit = I.pending != 0;
    const bool avg = I.use_avg != 0;
    const double ca = I.ca, cb = I.cb, beta = I.beta, etak = I.eta_k;
    const double tau = I.eta / I.omega;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = j0 + u * NT;
      if (j >= j1) break;
      double xv = (double)x[u];
      double gty = (double)g[u];
      if (commit) {
        const double xhv = (double)xh[u];
        const double ghv = (double)gh[u];
        xv = (double)(T)(ca * ((1.0 + beta) * xhv - beta * xv) + cb * (double)xa[u]);
        gty = (double)(T)(ca * ((1.0 + beta) * ghv - beta * gty) + cb * (double)ga[u]);
        it.x[j] = (T)xv;
        it.gty[j] = (T)gty;
        if (avg) it.sx[j] = (T)((double)sx[u] + etak * xhv);
      }
      const double cv = (double)c[u];
      const double xn = (double)(T)clampd(xv - tau * (cv - gty), (double)lo[u], (double)hi[u]);
      it.xh[j] = (T)xn;
      const double dx = xn - xv;
      acc[0] += dx * dx;
      acc[1] += cv * xn;
    }
  }
};

template <typename T, int U>
__device__ __forceinline__ void primal_body(int b, const Ranges& R, const IterPtrs<T>& it, const DataPtrs<T>& d,
                                            Inst* inst, int prec, double* rec) {
  __shared__ double lds[kWavesPerBlock * 2];
  const Inst& I = inst[R.blk_inst[b]];
  if (I.status != kActive || I.precision != prec) return;
  const bool commit = I.pending != 0, avg = commit && I.use_avg != 0;
  double acc[2] = {0.0, 0.0};
  const int j1 = R.blk_end[b];
  for (int j0 = R.blk_start[b] + (int)threadIdx.x; j0 < j1; j0 += U * kBlock) {
    PrimalElems<T, U> e;
    e.load(it, d, j0, j1, commit, avg);
    e.step(it, I, j0, j1, acc);
  }
  block_sum_store<2>(acc, lds, rec + (size_t)b * 2);
}

// The primal pass of every trial but the first of a chunk, with the reflection
// parameter of the trial before folded in.
template <typename T, bool IDLE>
__global__ __launch_bounds__(kBlock) void k_primal_fold(Ranges R, IterPtrs<T> it, DataPtrs<T> d, FoldIn f, int prec,
                                                        double* __restrict__ rec) {
  __shared__ double lds[kWavesPerBlock * 2];
  __shared__ Inst S;
  const int b = blockIdx.x, iid = R.blk_inst[b];
  const int j1 = R.blk_end[b];
  int j0 = R.blk_start[b] + (int)threadIdx.x;
  if (fold_idle<IDLE>(f, iid, prec)) {
    fold_pass_on(f, iid, prec, b == R.inst_blk0[iid]);
    return;
  }
  FoldBeta fold;
  fold.load(f, iid, &S);
  PrimalElems<T, kElems> e;
  e.load(it, d, min(j0, j1 - 1), j1, true, true);
  fold.decide(f, iid, &S, prec, b == R.inst_blk0[iid]);
  if (S.status != kActive || S.precision != prec) return;
  const bool commit = S.pending != 0, avg = commit && S.use_avg != 0;
  double acc[2] = {0.0, 0.0};
  if (j0 < j1) e.step(it, S, j0, j1, acc);
  for (j0 += kElems * kBlock; j0 < j1; j0 += kElems * kBlock) {
    e.load(it, d, j0, j1, commit, avg);
    e.step(it, S, j0, j1, acc);
  }
  block_sum_store<2>(acc, lds, rec + (size_t)b * 2);
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_primal(Ranges R, IterPtrs<T> it, DataPtrs<T> d,
                                                   Inst* __restrict__ inst, int prec,
                                                   double* __restrict__ rec) {
  primal_body<T, kElems>(blockIdx.x, R, it, d, inst, prec, rec);
}

// K1: CSR SpMV G x_hat with the fused dual step.  Record: ||dy||^2,
// dy^T G dx, ||(G x_hat - h) - Proj_Kd*(.)||^2, h^T y_hat.
template <typename T>
struct DualRow {  // a row's operands
  T y, gx, yh, gh, ya, ga, sy, h;
};
template <typename T>
struct DualEpilogue {
  IterPtrs<T> it;
  DataPtrs<T> d;
  bool commit, avg;
  double ca, cb, beta, etak, sigma;
  int mz_end, soc_start;
  __device__ __forceinline__ DualRow<T> load(int r) const {
    DualRow<T> o;
    o.y = it.y[r], o.gx = it.gx[r], o.h = d.h[r];
    if (commit) o.yh = it.yh[r], o.gh = it.gxh[r], o.ya = it.ya[r], o.ga = it.gxa[r];
    if (commit && avg) o.sy = it.sy[r];
    return o;
  }
  __device__ __forceinline__ void operator()(int r, double s, const DualRow<T>& o, double (&acc)[4]) const {
    double y = (double)o.y;
    double gx = (double)o.gx;
    if (commit) {
      const double yh = (double)o.yh;
      const double gh = (double)o.gh;
      y = (double)(T)(ca * ((1.0 + beta) * yh - beta * y) + cb * (double)o.ya);
      gx = (double)(T)(ca * ((1.0 + beta) * gh - beta * gx) + cb * (double)o.ga);
      it.y[r] = (T)y;
      it.gx[r] = (T)gx;
      if (avg) it.sy[r] = (T)((double)o.sy + etak * yh);
    }
    const double hv = (double)o.h;
    const double gxn = (double)(T)s;
    const double v = y + sigma * (hv - 2.0 * gxn + gx);
    if (r >= soc_start) {  // cone block row: projected with its block afterwards
      it.yh[r] = (T)v;
      it.gxh[r] = (T)gxn;
      return;
    }
    const bool zero_row = r < mz_end;
    const double yn = (double)(T)(zero_row ? v : fmax(v, 0.0));
    it.yh[r] = (T)yn;
    it.gxh[r] = (T)gxn;
    const double dy = yn - y;
    acc[0] += dy * dy;
    acc[1] += dy * (gxn - gx);
    const double res = gxn - hv;
    const double pr = zero_row ? res : fmin(res, 0.0);
    acc[2] += pr * pr;
    acc[3] += hv * yn;
  }
};

template <typename T>
__device__ __forceinline__ DualEpilogue<T> make_dual_epilogue(const Inst& I, const IterPtrs<T>& it,
                                                              const DataPtrs<T>& d) {
  DualEpilogue<T> e;
  e.it = it;
  e.d = d;
  e.commit = I.pending != 0;
  e.avg = I.use_avg != 0;
  e.ca = I.ca;
  e.cb = I.cb;
  e.beta = I.beta;
  e.etak = I.eta_k;
  e.sigma = I.eta * I.omega;
  e.mz_end = I.row0 + I.m_zero;
  e.soc_start = I.soc_start;
  return e;
}

template <typename T>
struct LamCol {  // a column's operands
  T c, l, u;
};
template <typename T>
__device__ __forceinline__ LamCol<T> lam_load(int j, const DataPtrs<T>& d) {
  return LamCol<T>{d.c[j], d.l[j], d.u[j]};
}

template <typename T>
__device__ __forceinline__ void lam_epilogue(int j, double s, const IterPtrs<T>& it, const LamCol<T>& o,
                                             double (&acc)[3]) {
  const double g = (double)(T)s;
  it.gtyh[j] = (T)g;
  const double lam = (double)o.c - g;
  const double lo = (double)o.l, hi = (double)o.u;
  const bool lf = isfinite(lo), uf = isfinite(hi);
  double res;
  if (!lf && !uf) res = lam;
  else if (!lf) res = fmax(lam, 0.0);
  else if (!uf) res = fmin(lam, 0.0);
  else res = 0.0;
  acc[0] += res * res;
  if (lf) acc[1] += lo * fmax(lam, 0.0);
  if (uf) acc[2] += hi * fmax(-lam, 0.0);
}

template <typename T, typename TM>
__device__ __forceinline__ void dual_body(int b, const RowBlocks& rb, const MatPtrs<TM>& A, const IterPtrs<T>& it,
                                          const DataPtrs<T>& d, Inst* inst, int prec, double* rec) {
  __shared__ double lds[kRowBlockCap + kWavesPerBlock * 4];
  const Inst& I = inst[rb.blk_inst[b]];
  if (I.status != kActive || I.precision != prec) return;
  const DualEpilogue<T> epi = make_dual_epilogue(I, it, d);
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  const T* const xs[1] = {it.xh};
  block_rows<1>(rb.blk_row0[b], rb.blk_row1[b], A.ptr, A.idx, A.val, xs, lds,
                [&](int r) { return epi.load(r); },
                [&](int r, const double* s, const DualRow<T>& o) { epi(r, s[0], o, acc); });
  __syncthreads();
  block_sum_store<4>(acc, lds, rec + (size_t)b * 4);
}

template <typename T, typename TM>
__global__ __launch_bounds__(kBlock) void k_dual(RowBlocks rb, MatPtrs<TM> A, IterPtrs<T> it,
                                                 DataPtrs<T> d, Inst* __restrict__ inst, int prec,
                                                 double* __restrict__ rec) {
  dual_body<T, TM>(blockIdx.x, rb, A, it, d, inst, prec, rec);
}

// ---------------------------------------------------------------------------
// Band-tile SpMV for single large instances (layout: BandTiles).  The gathers
// of a band-tile stay inside one window of the gathered vector, held in the L2
// of the XCDs that serve the window, and since the entries are sorted by
// gathered index the 64 lanes of a wave instruction read few cache lines.  Each
// wave sums its band in a private LDS array with plain read-modify-writes: the
// host never lets two entries of one 64-entry group share a slot, and LDS
// operations of one wave complete in issue order, so no atomics are needed and
// the result does not depend on scheduling.  The entry stream is software
// pipelined: packed entries and values are loaded two iterations ahead and the
// gathers one iteration ahead of the accumulation.  Output: part[panel * R + r].
// What bounds it: the L2's rate of gathered sectors (m = 2e5, n = 5e5, nnz = 5e6:
// 5e6 sectors of 64 B in 22 us, 14.5 TB/s; more waves per CU, with shorter bands
// or bands shared by several waves, bring more distinct sectors and no time, and
// staging x through LDS moves as many bytes through the same L2), and on the
// largest problems the stream of entries.  The LDS of a launch holds what its
// tallest tile uses, so that workgroups of short bands share a CU.
// ---------------------------------------------------------------------------
// Instances a check or evaluation pass works on.
// kModeRay: the infeasibility rays of a check, FP64 vectors whatever the
// instance's iterate precision.
enum Mode : int { kModeCheck = 0, kModeEvalStart = 1, kModeEvalFinal = 2, kModeRay = 3 };

__device__ __forceinline__ bool mode_selects(const Inst& I, int mode) {
  if (mode == kModeCheck) return I.status == kActive && I.check_due != 0;
  if (mode == kModeEvalStart) return I.status == kActive;
  if (mode == kModeRay) return I.status == kActive && I.check_due != 0 && I.ray_due != 0;
  return I.status == kDone && I.exit_code != 0;
}

// Precision filter of the check products: the ray pass serves every instance.
__device__ __forceinline__ bool prec_selects(const Inst& I, int mode, int prec) {
  return mode == kModeRay || I.precision == prec;
}

// What a band-tile accumulates per row.
struct SumProduct {
  template <typename TA>
  static __device__ __forceinline__ TA term(TA a, TA v, TA x) { return a + v * x; }
  template <typename TA>
  static __device__ __forceinline__ TA join(TA a, TA b) { return a + b; }
};
struct MaxProduct {  // of magnitudes, x >= 0
  static __device__ __forceinline__ double term(double a, double v, double x) { return fmax(a, fabs(v) * x); }
  static __device__ __forceinline__ double join(double a, double b) { return fmax(a, b); }
};
struct SumSquares {
  static __device__ __forceinline__ double term(double a, double v, double x) { return a + (v * x) * (v * x); }
  static __device__ __forceinline__ double join(double a, double b) { return a + b; }
};

// One wave's band-tile t: sums (or what OP joins) over the tile's entries of each row r
// of val * x[col], values TV, gathered vector TX, accumulation and output TA.  put(r, s)
// takes those of rows r + k * kWave (while below t.nrows) of the tile.  skip() tells, once the first entries are under
// way, whether the tile is left out.
//
// What a tile pays besides its entries: the descriptor and the instance's state,
// the clearing of the slots, and at the end the rows' sums with their extra slots.
// The entries do not wait for the first two.  The end reads an entry per row with
// extra slots, the first requested before the sweep, and adds the slots (consecutive
// in LDS) of eight rows a lane side by side.  (When the extra slots were listed in memory
// and each lane followed its rows' lists, a row of 5000 entries kept its tile 33 us
// behind its last entry; the products of m = 6e4, n = 1.2e5, nnz = 9.6e5 took 13.1
// and 11.3 us in FP64 and take 11.5 and 10.6, G^T y at m = 2.5e5, n = 5e5,
// nnz = 1.35e7 58 and 53, at m = 2e5, n = 5e5, nnz = 5e6 G x 35.2 and 33.4.  A word
// for every row instead of the rows with extra slots alone costs 22 us on tiles of 8192
// rows.)
//
// Deeper requests are no help where it counts: with 40 to 47 loads in flight per wave
// the first of these took 10.5 us, but the last 36.1 and G x of the second 78 for 72,
// and 23 and 48 with all lanes of a gather at one address: the lines that the gathers
// touch bound them.
constexpr int kBandFold = 8;  // rows per lane and step of a tile's end
template <typename TV, typename TX, typename TA, class OP = SumProduct, class Skip, class Put>
__device__ __forceinline__ void band_tile_product(const BandTiles& bt, const BandTile& t, TA* a,
                                                  const TV* __restrict__ val, const TX* __restrict__ x,
                                                  Skip skip, Put put) {
  constexpr int U = kBandUnroll;
  constexpr int F = kBandFold;
  const int lane = threadIdx.x & (kWave - 1);
  const TX* xs = x + t.col0;
  const int nit = t.nit;
  const uint32_t* pp = bt.pk + t.start + lane;
  const TV* vp = val + t.start + lane;
  const uint2* fold = bt.fold + t.fold0;
  const int nr = t.nrows, nf = t.nfold;
  constexpr uint32_t kSlotMask = (1u << kBandSlotBits) - 1u;
  uint32_t pA[U], pB[U], pC[U];
  TV vA[U], vB[U], vC[U];
  TX xA[U], xB[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    pA[u] = pB[u] = pC[u] = 0u;
    vA[u] = vB[u] = vC[u] = TV(0);
    xA[u] = xB[u] = TX(0);
  }
  if (nit > 0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      pA[u] = __builtin_nontemporal_load(pp + u * kWave);
      vA[u] = __builtin_nontemporal_load(vp + u * kWave);
    }
  }
  if (nit > 1) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      pB[u] = __builtin_nontemporal_load(pp + (U + u) * kWave);
      vB[u] = __builtin_nontemporal_load(vp + (U + u) * kWave);
    }
  }
  uint2 f[F];
#pragma unroll
  for (int k = 0; k < F; ++k) f[k] = k * kWave + lane < nf ? fold[k * kWave + lane] : uint2{0u, 0u};
  if (skip()) return;
  // the sink slot of the padding is never read and stays uninitialized
  for (int i = lane; i < t.used; i += kWave) a[i] = TA(0);
  wave_lds_order();
  if (nit > 0) {
#pragma unroll
    for (int u = 0; u < U; ++u) xA[u] = xs[pA[u] >> kBandSlotBits];
  }
  for (int it = 0; it < nit; ++it) {
    if (it + 2 < nit) {
      const int off = (it + 2) * U * kWave;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        pC[u] = __builtin_nontemporal_load(pp + off + u * kWave);
        vC[u] = __builtin_nontemporal_load(vp + off + u * kWave);
      }
    }
    if (it + 1 < nit) {
#pragma unroll
      for (int u = 0; u < U; ++u) xB[u] = xs[pB[u] >> kBandSlotBits];
    }
    // (groups of kWave entries may meet in a slot, one lane's and then another's; the slots
    // are data, so the compiler has to keep these accesses in order for each lane's own sake)
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t sl = pA[u] & kSlotMask;
      a[sl] = OP::term(a[sl], (TA)vA[u], (TA)xA[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      pA[u] = pB[u];
      vA[u] = vB[u];
      xA[u] = xB[u];
      pB[u] = pC[u];
      vB[u] = vC[u];
    }
  }
  wave_lds_order();
  // a row's slot, then its extra slots in order
  for (int r = lane; r - lane < nf; r += F * kWave) {
    uint2 g[F];
#pragma unroll
    for (int k = 0; k < F; ++k) g[k] = r + (F + k) * kWave < nf ? fold[r + (F + k) * kWave] : uint2{0u, 0u};
    TA s[F];
    uint32_t most = 0;
#pragma unroll
    for (int k = 0; k < F; ++k) {
      s[k] = f[k].x ? a[f[k].x & 0xFFFFu] : TA(0);
      most = max(most, f[k].x >> 16);
    }
    constexpr uint32_t E = 4;
    for (uint32_t q = 0; __any(q < most); q += E) {
      TA e[F][E];
#pragma unroll
      for (int k = 0; k < F; ++k)
#pragma unroll
        for (uint32_t j = 0; j < E; ++j) e[k][j] = q + j < f[k].x >> 16 ? a[f[k].y + q + j] : TA(0);
#pragma unroll
      for (int k = 0; k < F; ++k)
#pragma unroll
        for (uint32_t j = 0; j < E; ++j)
          if (q + j < f[k].x >> 16) s[k] = OP::join(s[k], e[k][j]);
    }
#pragma unroll
    for (int k = 0; k < F; ++k) {
      if (f[k].x) a[f[k].x & 0xFFFFu] = s[k];
      f[k] = g[k];
    }
  }
  wave_lds_order();
  for (int r = lane; r - lane < nr; r += F * kWave) {
    TA s[F];
#pragma unroll
    for (int k = 0; k < F; ++k) s[k] = a[min(r + k * kWave, nr - 1)];
    put(r, s);
  }
}

// The tile's sums into its window's partial sums.
template <typename TA>
struct PutPart {
  TA* out;
  int nr;
  __device__ __forceinline__ PutPart(const BandTile& t, TA* part, int64_t R)
      : out(part + (size_t)t.panel * R + t.row0), nr(t.nrows) {}
  __device__ __forceinline__ void operator()(int r, const TA (&s)[kBandFold]) const {
#pragma unroll
    for (int k = 0; k < kBandFold; ++k)
      if (r + k * kWave < nr) out[r + k * kWave] = s[k];
  }
};

// Trial products (K1: G x_hat, K2: G^T y_hat) in the iterate precision T.
template <typename T>
__global__ __launch_bounds__(kWave) void k_band_spmv(BandTiles bt, const T* __restrict__ val,
                                                                  const T* __restrict__ x, T* __restrict__ part,
                                                                  int64_t R, const Inst* __restrict__ inst,
                                                                  int prec, int need_acc, int idle) {
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];
  const BandTile t = bt.slot[blockIdx.x];  // (an idle slot has no entries and no rows)
  const auto skip = [&] {
    if (!inst) return false;
    // solver passes: only instances iterating in this precision (and accepted, for G^T y)
    const Inst& I = inst[t.inst];
    return I.status != kActive || I.precision != prec || (need_acc && I.last_acc == 0);
  };
  if (idle && skip()) return;  // (as fold_idle: before the first entries are requested)
  band_tile_product<T, T, T>(bt, t, reinterpret_cast<T*>(dyn), val, x, skip, PutPart<T>(t, part, R));
}

// Check / evaluation products with FP64 values of vectors in the iterate
// precision TX (which = 1: the average candidate, skipped where unused).
template <typename TX>
__global__ __launch_bounds__(kWave) void k_band_cand(BandTiles bt, const double* __restrict__ val,
                                                                  const TX* __restrict__ x,
                                                                  double* __restrict__ part, int64_t R,
                                                                  const Inst* __restrict__ inst, int prec, int mode,
                                                                  int which) {
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];
  const BandTile t = bt.slot[blockIdx.x];  // (an idle slot has no entries and no rows)
  const auto skip = [&] {
    const Inst& I = inst[t.inst];
    return !mode_selects(I, mode) || !prec_selects(I, mode, prec) ||
           (which == 1 && mode == kModeCheck && I.use_avg == 0);
  };
  if (skip()) return;  // (once a check: its launches for instances without work cost more than the wait)
  band_tile_product<double, TX, double>(bt, t, reinterpret_cast<double*>(dyn), val, x, [] { return false; },
                                        PutPart<double>(t, part, R));
}

// Window sums of the check / evaluation products (G^T y, then G x), per instance;
// a side without workgroups or without a vector is left out.
struct CombineSide {
  Ranges Rg;
  int P;
  int64_t R;
  const double *part0, *part1;
  double *out0, *out1;
};

__global__ __launch_bounds__(kBlock) void k_band_combine2(CombineSide cols, CombineSide rows,
                                                          const Inst* __restrict__ inst, int mode) {
  const bool first = (int)blockIdx.x < cols.Rg.nblk;
  const int b = first ? (int)blockIdx.x : (int)blockIdx.x - cols.Rg.nblk;
  const CombineSide& q = first ? cols : rows;
  const Inst& I = inst[q.Rg.blk_inst[b]];
  if (!mode_selects(I, mode)) return;
  const bool two = q.part1 != nullptr && (mode != kModeCheck || I.use_avg != 0);
  const int r1 = q.Rg.blk_end[b];
  for (int r = q.Rg.blk_start[b] + (int)threadIdx.x; r < r1; r += kBlock) {
    double s0 = 0.0, s1 = 0.0;
    for (int p = 0; p < q.P; ++p) {
      s0 += q.part0[(size_t)p * q.R + r];
      if (two) s1 += q.part1[(size_t)p * q.R + r];
    }
    q.out0[r] = s0;
    if (two) q.out1[r] = s1;
  }
}

// Sum of the P window partial sums per row (plain product of the band layout).
template <typename T>
__global__ void k_band_sum(const T* __restrict__ part, int P, int64_t R, T* __restrict__ out) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= R) return;
  double s = 0.0;
  for (int p = 0; p < P; ++p) s += (double)part[(size_t)p * R + r];
  out[r] = (T)s;
}

// Set-up: band-tile values from the scaled CSR (CSC) values.
__global__ void k_band_vals(const int32_t* __restrict__ src, int64_t n, const double* __restrict__ v64,
                            double* __restrict__ o64, float* __restrict__ o32) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  const int32_t q = src[e];
  const double v = q >= 0 ? v64[q] : 0.0;
  o64[e] = v;
  o32[e] = (float)v;
}

// s[u] += the P window partial sums of element e0 + u kBlock (the last one, end - 1,
// in place of those past it), in window order; two windows' loads in flight.
template <typename T, int U>
__device__ __forceinline__ void window_sums(const T* __restrict__ part, int P, int64_t M, int e0, int end,
                                            double (&s)[U]) {
  int p = 0;
  for (; p + 2 <= P; p += 2) {
    T v[2][U];
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int u = 0; u < U; ++u) v[k][u] = part[(size_t)(p + k) * M + min(e0 + u * kBlock, end - 1)];
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int u = 0; u < U; ++u) s[u] += (double)v[k][u];
  }
  if (p < P) {
    T v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = part[(size_t)p * M + min(e0 + u * kBlock, end - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u) s[u] += (double)v[u];
  }
}

// K1b: combine the P partial sums of G x_hat per row, then the dual step
// (same epilogue and record as k_dual).
template <typename T>
__global__ __launch_bounds__(kBlock) void k_dual_epi(Ranges R, const T* __restrict__ part, int P,
                                                     int64_t M, IterPtrs<T> it, DataPtrs<T> d,
                                                     const double* __restrict__ D1, Inst* __restrict__ inst,
                                                     int prec, double* __restrict__ rec) {
  __shared__ double lds[kWavesPerBlock * 4];
  const int b = blockIdx.x;
  const Inst& I = inst[R.blk_inst[b]];
  if (I.status != kActive || I.precision != prec) return;
  const DualEpilogue<T> epi = make_dual_epilogue(I, it, d);
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  const int r1 = R.blk_end[b];
  for (int q0 = R.blk_start[b] + (int)threadIdx.x; q0 < r1; q0 += kElems * kBlock) {
    DualRow<T> o[kElems];
    double s[kElems];
#pragma unroll
    for (int u = 0; u < kElems; ++u) {
      o[u] = epi.load(min(q0 + u * kBlock, r1 - 1));
      s[u] = 0.0;
    }
    window_sums<T, kElems>(part, P, M, q0, r1, s);
#pragma unroll
    for (int u = 0; u < kElems; ++u)
      if (q0 + u * kBlock < r1) epi(q0 + u * kBlock, s[u], o[u], acc);
  }
  if (R.blk_soc0 && R.blk_soc1[b] > R.blk_soc0[b]) {
    __syncthreads();  // the blocks' unprojected values and committed iterates are in memory
    // task 0: y_hat = Proj onto diag(1/D1) of the block's dual cone of the
    // stored value, with the line-search terms; task 1: the primal residual
    // of the reflection parameter, (G x_hat - h) against diag(D1) of the
    // block's cone (independent: task 1 reads neither y nor y_hat)
    // (the terms go through scalars: acc itself, written from the lambdas,
    // would be kept in scratch memory)
    double t0 = 0.0, t1 = 0.0, t2 = 0.0, t3 = 0.0;
    for_cone_tasks<2>(R, b, [&](auto who, int r0, int dim, int kind, int pass) {
      const bool dual = pass == 0;
      proj_cone(
          who, kind, dual, dim,
          [&](int i) { return dual ? (double)it.yh[r0 + i] : (double)it.gxh[r0 + i] - (double)d.h[r0 + i]; },
          [&](int i) { return dual ? 1.0 / D1[r0 + i] : D1[r0 + i]; },
          [&](int i, double p) {
            const int r = r0 + i;
            if (dual) {
              const double yn = (double)(T)p;
              it.yh[r] = (T)yn;
              const double dy = yn - (double)it.y[r];
              t0 += dy * dy;
              t1 += dy * ((double)it.gxh[r] - (double)it.gx[r]);
              t3 += (double)d.h[r] * yn;
            } else {
              const double pr = ((double)it.gxh[r] - (double)d.h[r]) - p;
              t2 += pr * pr;
            }
          });
    });
    acc[0] += t0;
    acc[1] += t1;
    acc[2] += t2;
    acc[3] += t3;
  }
  block_sum_store<4>(acc, lds, rec + (size_t)b * 4);
}

// K2b: combine the P partial sums of G^T y_hat per column, then the dual-slack
// epilogue (same record as k_lam).
template <typename T>
__global__ __launch_bounds__(kBlock) void k_lam_epi(Ranges R, const T* __restrict__ part, int P,
                                                    int64_t N, IterPtrs<T> it, DataPtrs<T> d,
                                                    Inst* __restrict__ inst, int prec,
                                                    double* __restrict__ rec) {
  __shared__ double lds[kWavesPerBlock * 3];
  const int b = blockIdx.x;
  const Inst& I = inst[R.blk_inst[b]];
  if (I.status != kActive || I.precision != prec || I.last_acc == 0) return;
  double acc[3] = {0.0, 0.0, 0.0};
  const int j1 = R.blk_end[b];
  for (int q0 = R.blk_start[b] + (int)threadIdx.x; q0 < j1; q0 += kElems * kBlock) {
    LamCol<T> o[kElems];
    double s[kElems];
#pragma unroll
    for (int u = 0; u < kElems; ++u) {
      o[u] = lam_load<T>(min(q0 + u * kBlock, j1 - 1), d);
      s[u] = 0.0;
    }
    window_sums<T, kElems>(part, P, N, q0, j1, s);
#pragma unroll
    for (int u = 0; u < kElems; ++u)
      if (q0 + u * kBlock < j1) lam_epilogue<T>(q0 + u * kBlock, s[u], it, o[u], acc);
  }
  block_sum_store<3>(acc, lds, rec + (size_t)b * 3);
}

__global__ __launch_bounds__(kBlock) void k_fin_ls(const int32_t* __restrict__ iblk_p,
                                                   const double* __restrict__ rec_p,
                                                   const int32_t* __restrict__ iblk_d,
                                                   const double* __restrict__ rec_d,
                                                   Inst* __restrict__ inst) {
  fin_ls_body(blockIdx.x, iblk_p, rec_p, iblk_d, rec_d, inst);
}

// K2: transposed SpMV G^T y_hat over the columns with the dual-slack epilogue.
// Record: ||lam - Proj_Lambda lam||^2, sum l lam+, sum u lam- (finite bounds).
template <typename T, typename TM>
__device__ __forceinline__ void lam_body(int b, const RowBlocks& rb, const MatPtrs<TM>& AT, const IterPtrs<T>& it,
                                         const DataPtrs<T>& d, Inst* inst, int prec, double* rec) {
  __shared__ double lds[kRowBlockCap + kWavesPerBlock * 3];
  const Inst& I = inst[rb.blk_inst[b]];
  if (I.status != kActive || I.precision != prec || I.last_acc == 0) return;
  double acc[3] = {0.0, 0.0, 0.0};
  const T* const ys[1] = {it.yh};
  block_rows<1>(rb.blk_row0[b], rb.blk_row1[b], AT.ptr, AT.idx, AT.val, ys, lds,
                [&](int j) { return lam_load<T>(j, d); },
                [&](int j, const double* s, const LamCol<T>& o) { lam_epilogue<T>(j, s[0], it, o, acc); });
  __syncthreads();
  block_sum_store<3>(acc, lds, rec + (size_t)b * 3);
}

template <typename T, typename TM>
__global__ __launch_bounds__(kBlock) void k_lam(RowBlocks rb, MatPtrs<TM> AT, IterPtrs<T> it,
                                                DataPtrs<T> d, Inst* __restrict__ inst, int prec,
                                                double* __restrict__ rec) {
  lam_body<T, TM>(blockIdx.x, rb, AT, it, d, inst, prec, rec);
}

__global__ __launch_bounds__(kBlock) void k_fin_beta(const int32_t* __restrict__ iblk_l,
                                                     const double* __restrict__ rec_l,
                                                     Inst* __restrict__ inst) {
  fin_beta_body(blockIdx.x, iblk_l, rec_l, inst);
}

// k_lam with the line-search decision folded in.  The decision comes after the gathers, so
// that neither waits for the other; a rejected trial, which k_lam leaves at once, pays for
// the product here.  Of the solves measured 1.2% of the trials at most are rejected (m = 1e6
// power law 15 of 1280, a quarter of it 16 of 3000, 200 x 500 1 of 8832), and a trial saves
// two launches: 22.6 us for 26.8 at 2.8e5 nonzeros, 35.0 for 39.3 at 9.1e5.
template <typename T, typename TM, bool IDLE>
__global__ __launch_bounds__(kBlock) void k_lam_fold(RowBlocks rb, MatPtrs<TM> AT, IterPtrs<T> it, DataPtrs<T> d,
                                                     FoldIn f, int prec, double* __restrict__ rec) {
  __shared__ double lds[kRowBlockCap + kWavesPerBlock * 3];
  __shared__ Inst S;
  const int b = blockIdx.x, iid = rb.blk_inst[b];
  __shared__ FoldLds L;
  const bool first = b == rb.inst_blk0[iid];
  if (fold_idle<IDLE>(f, iid, prec)) {
    fold_pass_on(f, iid, prec, first);
    return;
  }
  FoldLs fold;
  fold.load(f, iid, &S);
  double acc[3] = {0.0, 0.0, 0.0};
  bool live = false;
  const T* const ys[1] = {it.yh};
  block_rows<1>(rb.blk_row0[b], rb.blk_row1[b], AT.ptr, AT.idx, AT.val, ys, lds,
                [&](int j) { return lam_load<T>(j, d); },
                [&] { fold.early(L, first); },
                [&] {
                  fold.decide(f, L, iid, &S, prec, first);
                  live = S.status == kActive && S.precision == prec && S.last_acc != 0;
                },
                [&](int j, const double* s, const LamCol<T>& o) {
                  if (live) lam_epilogue<T>(j, s[0], it, o, acc);
                });
  if (!live) return;
  __syncthreads();
  block_sum_store<3>(acc, lds, rec + (size_t)b * 3);
}

// k_lam_epi with the line-search decision folded in.
template <typename T, bool IDLE>
__global__ __launch_bounds__(kBlock) void k_lam_epi_fold(Ranges R, const T* __restrict__ part, int P, int64_t N,
                                                         IterPtrs<T> it, DataPtrs<T> d, FoldIn f, int prec,
                                                         double* __restrict__ rec) {
  __shared__ double lds[kWavesPerBlock * 3];
  __shared__ Inst S;
  const int b = blockIdx.x, iid = R.blk_inst[b];
  __shared__ FoldLds L;
  const bool first = b == R.inst_blk0[iid];
  if (fold_idle<IDLE>(f, iid, prec)) {
    fold_pass_on(f, iid, prec, first);
    return;
  }
  FoldLs fold;
  fold.load(f, iid, &S);
  double acc[3] = {0.0, 0.0, 0.0};
  const int j1 = R.blk_end[b];
  bool decided = false;
  for (int e0 = R.blk_start[b]; e0 < j1; e0 += kElems * kBlock) {
    const int q0 = e0 + (int)threadIdx.x;
    LamCol<T> o[kElems];
    double s[kElems];
#pragma unroll
    for (int u = 0; u < kElems; ++u) {
      o[u] = lam_load<T>(min(q0 + u * kBlock, j1 - 1), d);
      s[u] = 0.0;
    }
    if (!decided) fold.early(L, first);
    window_sums<T, kElems>(part, P, N, q0, j1, s);
    if (!decided) {
      fold.decide(f, L, iid, &S, prec, first);
      if (S.status != kActive || S.precision != prec || S.last_acc == 0) return;
      decided = true;
    }
#pragma unroll
    for (int u = 0; u < kElems; ++u)
      if (q0 + u * kBlock < j1) lam_epilogue<T>(q0 + u * kBlock, s[u], it, o[u], acc);
  }
  block_sum_store<3>(acc, lds, rec + (size_t)b * 3);
}

// The line-search decision by one wave: as FoldLs, in the same order.
template <int NV>
__device__ __forceinline__ void wave_records(const double* __restrict__ rec, int b0, int b1, double (&v)[NV]) {
  const int lane = threadIdx.x & (kWave - 1);
  double a[kWavesPerBlock][NV];
#pragma unroll
  for (int w = 0; w < kWavesPerBlock; ++w) {
    const int k0 = b0 + w * kWave + lane, k1 = k0 + kBlock;
#pragma unroll
    for (int i = 0; i < NV; ++i)
      a[w][i] = (k0 < b1 ? rec[(size_t)k0 * NV + i] : 0.0) + (k1 < b1 ? rec[(size_t)k1 * NV + i] : 0.0);
  }
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] = wave_sum(a[0][i]);
#pragma unroll
  for (int w = 1; w < kWavesPerBlock; ++w)
#pragma unroll
    for (int i = 0; i < NV; ++i) v[i] += wave_sum(a[w][i]);
}

__device__ __forceinline__ void wave_decide(const FoldIn& f, int iid, Inst* S, double* pf, int prec, bool first) {
  const int lane = threadIdx.x & (kWave - 1);
  for (int i = lane; i < kInstWords; i += kWave)
    reinterpret_cast<uint64_t*>(S)[i] = reinterpret_cast<const uint64_t*>(f.in + iid)[i];
  double p[2], q[4];
  wave_records<2>(f.rec_a, f.iblk_a[iid], f.iblk_a[iid + 1], p);
  wave_records<4>(f.rec_b, f.iblk_b[iid], f.iblk_b[iid + 1], q);
  if (first && lane >= kWave - 2) {
    const int e = kWave - 1 - lane;
    pf[e] = pow((double)f.in[iid].kbar + 2.0, e ? -0.6 : -0.3);
  }
  __syncthreads();
  const bool mine = S->precision == prec;
  if (lane == 0 && S->status == kActive && mine) {
    const double f2[2] = {first ? pf[0] : 0.5, first ? pf[1] : 0.5};
    fin_ls_apply(*S, p, q, f2, first);
  }
  __syncthreads();
  if (first && mine)
    for (int i = lane; i < kInstWords; i += kWave)
      reinterpret_cast<uint64_t*>(f.out + iid)[i] = reinterpret_cast<const uint64_t*>(S)[i];
}

// G^T y_hat on band tiles of one window with the dual-slack epilogue at each tile's
// end (records per tile), the line-search decision of the trial folded in: every tile
// takes it under its first entries, and the launch's last workgroups, one per
// instance, write the records.  In place of the product's launch and k_lam_epi_fold's:
// a tile's end costs about 2 us more, the launch cost 9, and a rejected trial ends before
// its sweep.  (64 trials with 960 cone blocks 2430 -> 2310 us; 48 LPs of 1e3 to 2e4 rows
// 6910 -> 6680; m = 2e5, n = 5e5, nnz = 5e6 7450 -> 7310.)
template <typename T, bool IDLE>
__global__ __launch_bounds__(kWave) void k_band_lam_fold(BandTiles bt, const T* __restrict__ val, IterPtrs<T> it,
                                                         DataPtrs<T> d, FoldIn f, int prec, double* __restrict__ rec) {
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];
  __shared__ Inst S;
  __shared__ double pf[2];
  if ((int)blockIdx.x >= bt.nslot) {
    wave_decide(f, (int)blockIdx.x - bt.nslot, &S, pf, prec, true);
    return;
  }
  const BandTile t = bt.slot[blockIdx.x];
  if (t.tile < 0 || fold_idle<IDLE>(f, t.inst, prec)) return;
  bool live = false;
  double acc[3] = {0.0, 0.0, 0.0};
  const auto skip = [&] {
    wave_decide(f, t.inst, &S, pf, prec, false);
    live = S.status == kActive && S.precision == prec && S.last_acc != 0;
    return !live;
  };
  const auto put = [&](int r, const T(&s)[kBandFold]) {
    LamCol<T> o[kBandFold];
#pragma unroll
    for (int k = 0; k < kBandFold; ++k) o[k] = lam_load<T>(t.row0 + min(r + k * kWave, t.nrows - 1), d);
#pragma unroll
    for (int k = 0; k < kBandFold; ++k)
      if (r + k * kWave < t.nrows) lam_epilogue<T>(t.row0 + r + k * kWave, 0.0 + (double)s[k], it, o[k], acc);
  };
  band_tile_product<T, T, T>(bt, t, reinterpret_cast<T*>(dyn), val, (const T*)it.yh, skip, put);
  if (!live) return;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const double s = wave_sum(acc[i]);
    if ((threadIdx.x & (kWave - 1)) == 0) rec[(size_t)t.tile * 3 + i] = s;
  }
}

// A chunk of K trials of one instance per workgroup (small instances, row
// blocks): the passes of k_primal, k_dual, k_fin_ls, k_lam and k_fin_beta in
// order over the instance's blocks, separated by workgroup barriers instead
// of kernel boundaries.  All waves of the workgroup share one CU and its L1,
// so a barrier makes every global write of the previous pass visible.  The
// decisions are read from the instance record after each barrier, the same
// for every thread, so every barrier is reached by the whole workgroup.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_trials_wg(Ranges vcol, RowBlocks brow, RowBlocks bcol, MatPtrs<T> A,
                                                      MatPtrs<T> AT, IterPtrs<T> it, DataPtrs<T> d,
                                                      Inst* __restrict__ inst, int prec, double* rec_p,
                                                      double* rec_d, double* rec_l, int K) {
  const int iid = blockIdx.x;
  const int p0 = vcol.inst_blk0[iid], p1 = vcol.inst_blk0[iid + 1];
  const int d0 = brow.inst_blk0[iid], d1 = brow.inst_blk0[iid + 1];
  const int l0 = bcol.inst_blk0[iid], l1 = bcol.inst_blk0[iid + 1];
  for (int s = 0; s < K; ++s) {
    {
      const Inst& I = inst[iid];
      if (I.status != kActive || I.precision != prec) break;
    }
    for (int b = p0; b < p1; ++b) primal_body<T, kElems>(b, vcol, it, d, inst, prec, rec_p);
    __syncthreads();
    for (int b = d0; b < d1; ++b) dual_body<T, T>(b, brow, A, it, d, inst, prec, rec_d);
    __syncthreads();
    fin_ls_body(iid, vcol.inst_blk0, rec_p, brow.inst_blk0, rec_d, inst);
    __syncthreads();
    for (int b = l0; b < l1; ++b) lam_body<T, T>(b, bcol, AT, it, d, inst, prec, rec_l);
    __syncthreads();
    fin_beta_body(iid, bcol.inst_blk0, rec_l, inst);
    __syncthreads();
  }
}

// Row-wise passes of the LDS-resident chunk kernel (instances whose rows and
// columns hold at most kLdsRowMax entries), by kRowThreads threads: a few lanes per
// row of G (dual step) or of G^T (dual slack), the dot product in FP64, and one
// record for the whole instance.  A trial is five such steps, each bound by its
// chain of LDS reads, sums and barriers: 1.2 + 1.9 + 0.7 + 1.2 + 1.1 us at m = 200,
// n = 500, 2500 nonzeros with 256 threads and one per row.  40 trials there: 262 us
// with 256 threads, 242 with 512, 304 with 1024 (whose sums and barriers take more
// than the shorter rounds save).
constexpr int kRowThreads = 512;

// Lanes per row of a row-wise pass over `rows` rows by NT threads: as many as
// there are threads for, at most 8.
template <int NT>
__device__ __forceinline__ int row_lanes(int rows) {
  int L = 1;
  while (L < 8 && 2 * L * rows <= NT) L *= 2;
  return L;
}

// Entries [q0, q1) of a row against x by L lanes, this one the li-th; four entries of
// a lane in flight, the last up to three in one clamped step.  Every lane of the
// row gets the sum.
template <typename T>
__device__ __forceinline__ double row_dot_lanes(int q0, int q1, int L, int li, const int32_t* idx, const T* val,
                                                const T* x) {
  double s = 0.0;
  int q = q0 + li;
  for (; q + 3 * L < q1; q += 4 * L) {
    int c[4];
    double v[4], g[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      c[u] = idx[q + u * L];
      v[u] = (double)val[q + u * L];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) g[u] = (double)x[c[u]];
#pragma unroll
    for (int u = 0; u < 4; ++u) s += v[u] * g[u];
  }
  if (q < q1) {
    int c[3];
    double v[3], g[3];
#pragma unroll
    for (int u = 0; u < 3; ++u) {
      const int k = min(q + u * L, q1 - 1);
      c[u] = idx[k];
      v[u] = (double)val[k];
    }
#pragma unroll
    for (int u = 0; u < 3; ++u) g[u] = (double)x[c[u]];
#pragma unroll
    for (int u = 0; u < 3; ++u)
      if (q + u * L < q1) s += v[u] * g[u];
  }
  for (int off = L >> 1; off > 0; off >>= 1) s += __shfl_xor(s, off, kWave);
  return s;
}

template <typename T, int NT>
__device__ __forceinline__ void primal_elems_lds(int c0, int c1, const IterPtrs<T>& it, const DataPtrs<T>& d,
                                                 const Inst& I, double* rec) {
  __shared__ double lds[NT / kWave * 2];
  if (I.status != kActive) return;
  const bool commit = I.pending != 0, avg = commit && I.use_avg != 0;
  double acc[2] = {0.0, 0.0};
  for (int j = c0 + (int)threadIdx.x; j < c1; j += NT) {
    PrimalElems<T, 1, NT> e;
    e.load(it, d, j, c1, commit, avg);
    e.step(it, I, j, c1, acc);
  }
  block_sum_store<2, NT / kWave>(acc, lds, rec);
}

template <typename T, int NT>
__device__ __forceinline__ void dual_rows_lds(int r0, int r1, const MatPtrs<T>& A, const IterPtrs<T>& it,
                                              const DataPtrs<T>& d, const Inst& I, double* rec) {
  __shared__ double lds[NT / kWave * 4];
  if (I.status != kActive) return;
  const DualEpilogue<T> epi = make_dual_epilogue(I, it, d);
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  const int L = row_lanes<NT>(r1 - r0), li = threadIdx.x & (L - 1);
  for (int r = r0 + (int)threadIdx.x / L; r < r1; r += NT / L) {
    const DualRow<T> o = epi.load(r);
    const double s = row_dot_lanes(A.ptr[r], A.ptr[r + 1], L, li, A.idx, A.val, it.xh);
    if (li == 0) epi(r, s, o, acc);
  }
  block_sum_store<4, NT / kWave>(acc, lds, rec);
}

template <typename T, int NT>
__device__ __forceinline__ void lam_rows_lds(int c0, int c1, const MatPtrs<T>& AT, const IterPtrs<T>& it,
                                             const DataPtrs<T>& d, const Inst& I, double* rec) {
  __shared__ double lds[NT / kWave * 3];
  if (I.status != kActive || I.last_acc == 0) return;
  double acc[3] = {0.0, 0.0, 0.0};
  const int L = row_lanes<NT>(c1 - c0), li = threadIdx.x & (L - 1);
  for (int j = c0 + (int)threadIdx.x / L; j < c1; j += NT / L) {
    const LamCol<T> o = lam_load<T>(j, d);
    const double s = row_dot_lanes(AT.ptr[j], AT.ptr[j + 1], L, li, AT.idx, AT.val, it.yh);
    if (li == 0) lam_epilogue<T>(j, s, it, o, acc);
  }
  block_sum_store<3, NT / kWave>(acc, lds, rec);
}

template <typename T>
__device__ __forceinline__ void lds_copy(T* __restrict__ dst, const T* __restrict__ src, int64_t n) {
  for (int64_t i = threadIdx.x; i < n; i += blockDim.x) dst[i] = src[i];
}

// k_trials_wg with the instance resident in LDS: the kernel copies its
// iterates, data, matrix rows and columns, schedule tables and Inst record
// into LDS, runs the chunk's K trials there (pointers into LDS, offset so that
// the device functions keep using global indices), then writes back what the
// trials change.  Every dependent step of a trial is then an LDS access
// instead of an HBM round trip.  The host launches it only when the largest
// instance fits (dynamic LDS of lds_layout(...).total bytes).
template <typename T, int NT>
__global__ __launch_bounds__(NT) void k_trials_lds(Ranges vcol, RowBlocks brow, RowBlocks bcol, MatPtrs<T> A,
                                                   MatPtrs<T> AT, IterPtrs<T> it, DataPtrs<T> d,
                                                   Inst* __restrict__ inst, int prec, int K) {
  constexpr bool rowwise = NT > kBlock;
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];
  __shared__ Inst Ish;
  __shared__ int32_t iblk[6];
  const int iid = blockIdx.x;
  {
    const uint64_t* s = reinterpret_cast<const uint64_t*>(&inst[iid]);
    uint64_t* t = reinterpret_cast<uint64_t*>(&Ish);
    for (int i = threadIdx.x; i < (int)(sizeof(Inst) / 8); i += NT) t[i] = s[i];
    if (threadIdx.x == 0) {
      iblk[0] = vcol.inst_blk0[iid];
      iblk[1] = vcol.inst_blk0[iid + 1];
      iblk[2] = brow.inst_blk0[iid];
      iblk[3] = brow.inst_blk0[iid + 1];
      iblk[4] = bcol.inst_blk0[iid];
      iblk[5] = bcol.inst_blk0[iid + 1];
    }
  }
  __syncthreads();
  if (Ish.status != kActive || Ish.precision != prec || K < 1) return;
  const int r0 = Ish.row0, m = Ish.rows, c0 = Ish.col0, n = Ish.cols;
  const int p0 = iblk[0], np = iblk[1] - p0, d0 = iblk[2], nd = iblk[3] - d0, l0 = iblk[4], nl = iblk[5] - l0;
  const int q0 = A.ptr[r0], nnz = A.ptr[r0 + m] - q0;
  const int t0 = AT.ptr[c0];
  const LdsLayout L = lds_layout(m, n, nnz, np, nd, nl, sizeof(T));
  T* vec = reinterpret_cast<T*>(dyn + L.vec);
  T* dat = reinterpret_cast<T*>(dyn + L.dat);
  // iterates (x-like: n values each, then y-like: m values each)
  T* const xs[7] = {it.x, it.xa, it.xh, it.gty, it.gtya, it.gtyh, it.sx};
  T* const ys[7] = {it.y, it.ya, it.yh, it.gx, it.gxa, it.gxh, it.sy};
  for (int v = 0; v < 7; ++v) lds_copy(vec + (size_t)v * n, xs[v] + c0, n);
  for (int v = 0; v < 7; ++v) lds_copy(vec + (size_t)7 * n + (size_t)v * m, ys[v] + r0, m);
  lds_copy(dat, d.c + c0, n);
  lds_copy(dat + n, d.l + c0, n);
  lds_copy(dat + 2 * n, d.u + c0, n);
  lds_copy(dat + 3 * n, d.h + r0, m);
  int32_t* rp = reinterpret_cast<int32_t*>(dyn + L.rp);
  int32_t* ci = reinterpret_cast<int32_t*>(dyn + L.ci);
  T* va = reinterpret_cast<T*>(dyn + L.va);
  int32_t* cp = reinterpret_cast<int32_t*>(dyn + L.cp);
  int32_t* ri = reinterpret_cast<int32_t*>(dyn + L.ri);
  T* vt = reinterpret_cast<T*>(dyn + L.vt);
  lds_copy(rp, A.ptr + r0, m + 1);
  lds_copy(ci, A.idx + q0, nnz);
  lds_copy(va, A.val + q0, nnz);
  lds_copy(cp, AT.ptr + c0, n + 1);
  lds_copy(ri, AT.idx + t0, nnz);
  lds_copy(vt, AT.val + t0, nnz);
  double* recp = reinterpret_cast<double*>(dyn + L.rec);
  double* recd = recp + 2 * max(np, 1);
  double* recl = recd + 4 * max(nd, 1);
  int32_t* bt = reinterpret_cast<int32_t*>(dyn + L.blk);
  lds_copy(bt, vcol.blk_start + p0, np);
  lds_copy(bt + np, vcol.blk_end + p0, np);
  lds_copy(bt + 2 * np, vcol.blk_inst + p0, np);
  int32_t* bd = bt + 3 * np;
  lds_copy(bd, brow.blk_row0 + d0, nd);
  lds_copy(bd + nd, brow.blk_row1 + d0, nd);
  lds_copy(bd + 2 * nd, brow.blk_inst + d0, nd);
  int32_t* bl = bd + 3 * nd;
  lds_copy(bl, bcol.blk_row0 + l0, nl);
  lds_copy(bl + nl, bcol.blk_row1 + l0, nl);
  lds_copy(bl + 2 * nl, bcol.blk_inst + l0, nl);
  __syncthreads();
  // the same structures over LDS, indexed with global row, column, entry,
  // block and instance numbers
  IterPtrs<T> li = it;
  T* const lx[7] = {vec, vec + n, vec + 2 * n, vec + 3 * n, vec + 4 * n, vec + 5 * n, vec + 6 * n};
  T* const ly0 = vec + (size_t)7 * n;
  li.x = lx[0] - c0;
  li.xa = lx[1] - c0;
  li.xh = lx[2] - c0;
  li.gty = lx[3] - c0;
  li.gtya = lx[4] - c0;
  li.gtyh = lx[5] - c0;
  li.sx = lx[6] - c0;
  li.y = ly0 - r0;
  li.ya = ly0 + m - r0;
  li.yh = ly0 + 2 * m - r0;
  li.gx = ly0 + 3 * m - r0;
  li.gxa = ly0 + 4 * m - r0;
  li.gxh = ly0 + 5 * m - r0;
  li.sy = ly0 + 6 * m - r0;
  const DataPtrs<T> ld{dat - c0, dat + n - c0, dat + 2 * n - c0, dat + 3 * n - r0};
  const MatPtrs<T> LA{rp - r0, ci - q0, va - q0};
  const MatPtrs<T> LAT{cp - c0, ri - t0, vt - t0};
  Ranges lv = vcol;
  lv.blk_start = bt - p0;
  lv.blk_end = bt + np - p0;
  lv.blk_inst = bt + 2 * np - p0;
  lv.inst_blk0 = iblk - iid;
  RowBlocks lr = brow;
  lr.blk_row0 = bd - d0;
  lr.blk_row1 = bd + nd - d0;
  lr.blk_inst = bd + 2 * nd - d0;
  lr.inst_blk0 = iblk + 2 - iid;
  RowBlocks lc = bcol;
  lc.blk_row0 = bl - l0;
  lc.blk_row1 = bl + nl - l0;
  lc.blk_inst = bl + 2 * nl - l0;
  lc.inst_blk0 = iblk + 4 - iid;
  Inst* li_inst = &Ish - iid;
  double* rp_ = recp - 2 * (size_t)p0;
  double* rd_ = recd - 4 * (size_t)d0;
  double* rl_ = recl - 3 * (size_t)l0;
  // Row-wise instances leave one record in each pass (one[] is the per-instance
  // block table of a single record); the others keep their blocks.
  __shared__ int32_t one[2];
  __shared__ double pf[2];
  if (threadIdx.x == 0) {
    one[0] = 0;
    one[1] = 1;
  }
  if (threadIdx.x == kWave) {  // line-search factors of the first trial
    const double kb = (double)Ish.kbar + 2.0;
    pf[0] = pow(kb, -0.3);
    pf[1] = pow(kb, -0.6);
  }
  __syncthreads();
  for (int s = 0; s < K; ++s) {
    if (Ish.status != kActive || Ish.precision != prec) break;
    if constexpr (rowwise) {
      primal_elems_lds<T, NT>(c0, c0 + n, li, ld, Ish, recp);
      __syncthreads();
      dual_rows_lds<T, NT>(r0, r0 + m, LA, li, ld, Ish, recd);
      __syncthreads();
      fin_ls_body(iid, one - iid, recp, one - iid, recd, li_inst, pf);
      __syncthreads();
      lam_rows_lds<T, NT>(c0, c0 + n, LAT, li, ld, Ish, recl);
      __syncthreads();
      fin_beta_body(iid, one - iid, recl, li_inst);
    } else {
      for (int b = p0; b < p0 + np; ++b) primal_body<T, 2>(b, lv, li, ld, li_inst, prec, rp_);
      __syncthreads();
      for (int b = d0; b < d0 + nd; ++b) dual_body<T, T>(b, lr, LA, li, ld, li_inst, prec, rd_);
      __syncthreads();
      fin_ls_body(iid, lv.inst_blk0, rp_, lr.inst_blk0, rd_, li_inst, pf);
      __syncthreads();
      for (int b = l0; b < l0 + nl; ++b) lam_body<T, T>(b, lc, LAT, li, ld, li_inst, prec, rl_);
      __syncthreads();
      fin_beta_body(iid, lc.inst_blk0, rl_, li_inst);
    }
    // every thread has passed the finalizer's reductions; thread 0 may still be
    // in its scalar part (which does not touch kbar), while wave 1 forms the
    // next trial's line-search factors
    if (threadIdx.x == kWave) {
      const double kb = (double)Ish.kbar + 2.0;
      pf[0] = pow(kb, -0.3);
      pf[1] = pow(kb, -0.6);
    }
    __syncthreads();
  }
  // write back what trials change: x, x_hat, G^T y, G^T y_hat, S_x and the row
  // counterparts (anchors and data are read-only here), then the record
  const int wx[5] = {0, 2, 3, 5, 6};
  for (int v = 0; v < 5; ++v) {
    const T* src = vec + (size_t)wx[v] * n;
    T* dst = xs[wx[v]] + c0;
    for (int i = threadIdx.x; i < n; i += NT) dst[i] = src[i];
    const T* sy_ = ly0 + (size_t)wx[v] * m;
    T* dy_ = ys[wx[v]] + r0;
    for (int i = threadIdx.x; i < m; i += NT) dy_[i] = sy_[i];
  }
  {
    const uint64_t* s = reinterpret_cast<const uint64_t*>(&Ish);
    uint64_t* t = reinterpret_cast<uint64_t*>(&inst[iid]);
    for (int i = threadIdx.x; i < (int)(sizeof(Inst) / 8); i += NT) t[i] = s[i];
  }
}

// ===========================================================================
// Restart / termination check
// ===========================================================================

// The column and the row side of a step of a check or an evaluation depend on
// nothing of each other: one launch takes both, its first workgroups the columns.
// (Each of these launches is 4.7 us for a problem of a few hundred rows and 6 to 7
// for 2e4 x 4e4, 3e5 nonzeros: start-up, not traffic.)

// Apply the pending Halpern commit, then form the average candidate S / sum(eta).
template <typename T>
struct CommitSide {
  Ranges R;
  T* z;
  const T *zh, *za;
  T* g;
  const T *gh, *ga;
  T *s, *zbar;
};

template <typename T>
static CommitSide<T> commit_cols(const Ranges& R, const IterPtrs<T>& it) {
  return {R, it.x, it.xh, it.xa, it.gty, it.gtyh, it.gtya, it.sx, it.xbar};
}
template <typename T>
static CommitSide<T> commit_rows(const Ranges& R, const IterPtrs<T>& it) {
  return {R, it.y, it.yh, it.ya, it.gx, it.gxh, it.gxa, it.sy, it.ybar};
}

template <typename T>
__device__ __forceinline__ void commit_avg(int b, const CommitSide<T>& q, const Inst* __restrict__ inst, int prec) {
  const Ranges& R = q.R;
  T *__restrict__ z = q.z, *__restrict__ g = q.g, *__restrict__ s = q.s, *__restrict__ zbar = q.zbar;
  const T *__restrict__ zh = q.zh, *__restrict__ za = q.za, *__restrict__ gh = q.gh, *__restrict__ ga = q.ga;
  const Inst& I = inst[R.blk_inst[b]];
  if (I.status != kActive || I.check_due == 0 || I.precision != prec) return;
  const bool commit = I.pending != 0;
  const bool avg = I.use_avg != 0;
  const double ca = I.ca, cb = I.cb, beta = I.beta, etak = I.eta_k;
  const double inv_sum = 1.0 / I.sum_eta;
  const int j1 = R.blk_end[b];
  for (int j = R.blk_start[b] + (int)threadIdx.x; j < j1; j += kBlock) {
    const double zhv = (double)zh[j];
    double sv = avg ? (double)s[j] : 0.0;
    if (commit) {
      z[j] = (T)(ca * ((1.0 + beta) * zhv - beta * (double)z[j]) + cb * (double)za[j]);
      g[j] = (T)(ca * ((1.0 + beta) * (double)gh[j] - beta * (double)g[j]) + cb * (double)ga[j]);
      if (avg) {
        sv = (double)(T)(sv + etak * zhv);
        s[j] = (T)sv;
      }
    }
    if (avg) zbar[j] = (T)(sv * inv_sum);
  }
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_commit_avg(CommitSide<T> cols, CommitSide<T> rows,
                                                       const Inst* __restrict__ inst, int prec) {
  const int b = blockIdx.x;
  if (b < cols.R.nblk) commit_avg(b, cols, inst, prec);
  else commit_avg(b - cols.R.nblk, rows, inst, prec);
}

// Two products with one matrix pass: out0 = A in0, out1 = A in1 (FP64 values,
// FP64 output), of G^T and of G.  in1 may be null.  Selected instances only.
template <typename T>
struct Spmv2Side {
  RowBlocks rb;
  MatPtrs<double> A;
  const T *in0, *in1;
  double *out0, *out1;
};

template <typename T>
__global__ __launch_bounds__(kBlock) void k_spmv2(Spmv2Side<T> cols, Spmv2Side<T> rows, const Inst* __restrict__ inst,
                                                  int prec, int mode) {
  __shared__ double lds[2 * kRowBlockCap + kWavesPerBlock * 2];
  const bool first = (int)blockIdx.x < cols.rb.nblk;
  const int b = first ? (int)blockIdx.x : (int)blockIdx.x - cols.rb.nblk;
  const RowBlocks rb = first ? cols.rb : rows.rb;
  const MatPtrs<double> A = first ? cols.A : rows.A;
  const T *__restrict__ in0 = first ? cols.in0 : rows.in0, *__restrict__ in1 = first ? cols.in1 : rows.in1;
  double *__restrict__ out0 = first ? cols.out0 : rows.out0, *__restrict__ out1 = first ? cols.out1 : rows.out1;
  const Inst& I = inst[rb.blk_inst[b]];
  if (!mode_selects(I, mode) || !prec_selects(I, mode, prec)) return;
  const bool two = (in1 != nullptr) && (mode != kModeCheck || I.use_avg != 0);
  if (two) {
    const T* const xs[2] = {in0, in1};
    block_rows<2>(rb.blk_row0[b], rb.blk_row1[b], A.ptr, A.idx, A.val, xs, lds, [&](int r, const double* s) {
      out0[r] = s[0];
      out1[r] = s[1];
    });
  } else {
    const T* const xs[1] = {in0};
    block_rows<1>(rb.blk_row0[b], rb.blk_row1[b], A.ptr, A.idx, A.val, xs, lds,
                  [&](int r, const double* s) { out0[r] = s[0]; });
  }
}

// Candidate reductions over the columns.  Per candidate c (0: PDHG output or
// evaluated point, 1: average): sums ||x_c - x_a||^2, ||b1||^2, ||lam - Proj lam||^2,
// sum l lam+, sum u lam-, c^T x_c; maxima of the unscaled dual residual and |G^T y|.
// Record layout: [c0 sums(6), c1 sums(6), c0 max(2), c1 max(2)].
constexpr int kCandColsNV = 16, kCandColsNS = 12;
template <typename T>
__device__ __forceinline__ void cand_cols(int b, const Ranges& R, const T* x0, const T* x1, const T* xa,
                                          const double* g0, const double* g1, const DataPtrs<double>& d,
                                          const double* D2, const Inst* inst, int prec, int mode, double* rec) {
  __shared__ double lds[kWavesPerBlock * kCandColsNV];
  const Inst& I = inst[R.blk_inst[b]];
  if (!mode_selects(I, mode) || I.precision != prec) return;
  const int nc = (mode == kModeCheck && I.use_avg) ? 2 : 1;
  double acc[kCandColsNV];
#pragma unroll
  for (int i = 0; i < kCandColsNV; ++i) acc[i] = 0.0;
  const int j1 = R.blk_end[b];
  for (int j = R.blk_start[b] + (int)threadIdx.x; j < j1; j += kBlock) {
    const double c = d.c[j], lo = d.l[j], hi = d.u[j], dj = D2[j];
    const bool lf = isfinite(lo), uf = isfinite(hi);
    const double xav = (double)xa[j];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (q >= nc) break;
      const double xc = (double)(q == 0 ? x0[j] : x1[j]);
      const double gty = q == 0 ? g0[j] : g1[j];
      const double dxa = xc - xav;
      const double lam = c - gty;
      double res;
      if (!lf && !uf) res = lam;
      else if (!lf) res = fmax(lam, 0.0);
      else if (!uf) res = fmin(lam, 0.0);
      else res = 0.0;
      acc[q * 6 + 0] += dxa * dxa;
      acc[q * 6 + 1] += lam * lam;
      acc[q * 6 + 2] += res * res;
      if (lf) acc[q * 6 + 3] += lo * fmax(lam, 0.0);
      if (uf) acc[q * 6 + 4] += hi * fmax(-lam, 0.0);
      acc[q * 6 + 5] += c * xc;
      acc[12 + q * 2 + 0] = fmax(acc[12 + q * 2 + 0], fabs(res) / dj);
      acc[12 + q * 2 + 1] = fmax(acc[12 + q * 2 + 1], fabs(gty) / dj);
    }
  }
  block_summax_store<kCandColsNV, kCandColsNS>(acc, lds, rec + (size_t)b * kCandColsNV);
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_cand_cols(Ranges R, const T* __restrict__ x0,
                                                      const T* __restrict__ x1, const T* __restrict__ xa,
                                                      const double* __restrict__ g0,
                                                      const double* __restrict__ g1,
                                                      DataPtrs<double> d, const double* __restrict__ D2,
                                                      const Inst* __restrict__ inst, int prec, int mode,
                                                      double* __restrict__ rec) {
  cand_cols<T>(blockIdx.x, R, x0, x1, xa, g0, g1, d, D2, inst, prec, mode, rec);
}

// Candidate reductions over the rows: sums ||y_c - y_a||^2, ||b2||^2,
// ||(Gx-h) - Proj_Kd*||^2, h^T y_c; maxima of the unscaled primal residual,
// |G x| and |Proj_Kd*(G x - h)|.  Layout: [c0 sums(4), c1 sums(4), c0 max(3), c1 max(3)].
constexpr int kCandRowsNV = 14, kCandRowsNS = 8;
// CONES: the range may hold cone blocks (as in the other passes over rows).
template <typename T, bool CONES>
__device__ __forceinline__ void cand_rows(int b, const Ranges& R, const T* y0, const T* y1, const T* ya,
                                          const double* g0, const double* g1, const DataPtrs<double>& d,
                                          const double* D1, const Inst* inst, int prec, int mode, double* rec) {
  __shared__ double lds[kWavesPerBlock * kCandRowsNV];
  const Inst& I = inst[R.blk_inst[b]];
  if (!mode_selects(I, mode) || I.precision != prec) return;
  const int nc = (mode == kModeCheck && I.use_avg) ? 2 : 1;
  const int mz_end = I.row0 + I.m_zero;
  double acc[kCandRowsNV];
#pragma unroll
  for (int i = 0; i < kCandRowsNV; ++i) acc[i] = 0.0;
  const int i1 = R.blk_end[b];
  for (int i = R.blk_start[b] + (int)threadIdx.x; i < i1; i += kBlock) {
    if (i >= I.soc_start) continue;  // cone block rows: below
    const double h = d.h[i], di = D1[i];
    const double yav = (double)ya[i];
    const bool zero_row = i < mz_end;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (q >= nc) break;
      const double yc = (double)(q == 0 ? y0[i] : y1[i]);
      const double gx = q == 0 ? g0[i] : g1[i];
      const double dya = yc - yav;
      const double res = gx - h;
      const double pr = zero_row ? res : fmin(res, 0.0);
      const double proj = zero_row ? 0.0 : fmax(res, 0.0);
      acc[q * 4 + 0] += dya * dya;
      acc[q * 4 + 1] += res * res;
      acc[q * 4 + 2] += pr * pr;
      acc[q * 4 + 3] += h * yc;
      acc[8 + q * 3 + 0] = fmax(acc[8 + q * 3 + 0], fabs(pr) / di);
      acc[8 + q * 3 + 1] = fmax(acc[8 + q * 3 + 1], fabs(gx) / di);
      acc[8 + q * 3 + 2] = fmax(acc[8 + q * 3 + 2], proj / di);
    }
  }
  // cone blocks: the same terms, with the residual r = G x - h projected onto
  // diag(D1) of the block's cone for the scaled L2 term and, unscaled (r / D1),
  // onto the cone itself for the infinity-norm termination terms
  // (one task per block, candidate q and scaled / unscaled projection, spread
  // over the waves, with one inlined projection; the terms go through scalars
  // to acc)
  // per candidate: sums c[q][0..3] for acc[q*4 + i], maxima c[q][4..6] for acc[8 + q*3 + i - 4]
  if constexpr (CONES) {
    double c00 = 0.0, c01 = 0.0, c02 = 0.0, c03 = 0.0, c04 = 0.0, c05 = 0.0, c06 = 0.0;
    double c10 = 0.0, c11 = 0.0, c12 = 0.0, c13 = 0.0, c14 = 0.0, c15 = 0.0, c16 = 0.0;
    for_cone_tasks<2 * kMaxCand>(R, b, [&](auto who, int r0, int dim, int kind, int task) {
      const int q = task >> 1, pass = task & 1;
      if (who.any(q < nc)) {
        const T* yq = q == 0 ? y0 : y1;
        const double* gq = q == 0 ? g0 : g1;
        double t0 = 0.0, t1 = 0.0, t2 = 0.0, t3 = 0.0, t4 = 0.0, t5 = 0.0, t6 = 0.0;
        if (pass == 0) {
          for (int i = who.first(); i < who.count(dim); i += who.stride()) {
            const int r = r0 + i;
            const double yc = (double)yq[r], gx = gq[r], h = d.h[r];
            const double dya = yc - (double)ya[r], res = gx - h;
            t0 += dya * dya;
            t1 += res * res;
            t3 += h * yc;
            t5 = fmax(t5, fabs(gx) / D1[r]);
          }
        }
        const bool scaled = pass == 0;
        proj_cone(
            who, kind, false, dim,
            [&](int i) { return scaled ? gq[r0 + i] - d.h[r0 + i] : (gq[r0 + i] - d.h[r0 + i]) / D1[r0 + i]; },
            [&](int i) { return scaled ? D1[r0 + i] : 1.0; },
            [&](int i, double p) {
              if (scaled) {
                const double pr = (gq[r0 + i] - d.h[r0 + i]) - p;
                t2 += pr * pr;
              } else {
                const double ru = (gq[r0 + i] - d.h[r0 + i]) / D1[r0 + i];
                t4 = fmax(t4, fabs(ru - p));
                t6 = fmax(t6, fabs(p));
              }
            });
        if (q == 0) {
          c00 += t0, c01 += t1, c02 += t2, c03 += t3;
          c04 = fmax(c04, t4), c05 = fmax(c05, t5), c06 = fmax(c06, t6);
        } else {
          c10 += t0, c11 += t1, c12 += t2, c13 += t3;
          c14 = fmax(c14, t4), c15 = fmax(c15, t5), c16 = fmax(c16, t6);
        }
      }
    });
    acc[0] += c00, acc[1] += c01, acc[2] += c02, acc[3] += c03;
    acc[4] += c10, acc[5] += c11, acc[6] += c12, acc[7] += c13;
    acc[8] = fmax(acc[8], c04), acc[9] = fmax(acc[9], c05), acc[10] = fmax(acc[10], c06);
    acc[11] = fmax(acc[11], c14), acc[12] = fmax(acc[12], c15), acc[13] = fmax(acc[13], c16);
  }
  block_summax_store<kCandRowsNV, kCandRowsNS>(acc, lds, rec + (size_t)b * kCandRowsNV);
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_cand_rows(Ranges R, const T* __restrict__ y0,
                                                      const T* __restrict__ y1, const T* __restrict__ ya,
                                                      const double* __restrict__ g0,
                                                      const double* __restrict__ g1,
                                                      DataPtrs<double> d, const double* __restrict__ D1,
                                                      const Inst* __restrict__ inst, int prec, int mode,
                                                      double* __restrict__ rec) {
  cand_rows<T, true>(blockIdx.x, R, y0, y1, ya, g0, g1, d, D1, inst, prec, mode, rec);
}

// Combine the candidate reductions: radii, KKT errors, termination errors,
// and the start of the bisection (t0 = r / sqrt(tau|b1|^2 + sigma|b2|^2)).
__device__ __forceinline__ void cand_fin(int iid, const Ranges& rc, const double* rec_c, const Ranges& rr,
                                         const double* rec_r, Inst* inst, int mode) {
  __shared__ double lds[kWavesPerBlock * kCandColsNV];
  Inst& I = inst[iid];
  if (!mode_selects(I, mode)) return;
  double cs[kCandColsNV], rs[kCandRowsNV];
  reduce_records<kCandColsNV, kCandColsNS>(rec_c, rc.inst_blk0[iid], rc.inst_blk0[iid + 1], lds, cs);
  reduce_records<kCandRowsNV, kCandRowsNS>(rec_r, rr.inst_blk0[iid], rr.inst_blk0[iid + 1], lds, rs);
  if (threadIdx.x != 0) return;
  const int nc = (mode == kModeCheck && I.use_avg) ? 2 : 1;
  const double omega = I.omega;
  const double tau = I.eta_hat / omega, sigma = I.eta_hat * omega;
  for (int q = 0; q < nc; ++q) {
    CandState& C = I.cand[q];
    C.dxa2 = cs[q * 6 + 0];
    C.dya2 = rs[q * 4 + 0];
    const double b1sq = cs[q * 6 + 1], b2sq = rs[q * 4 + 1];
    C.errd = sqrt(cs[q * 6 + 2]);
    C.errp = sqrt(rs[q * 4 + 2]);
    C.pobj = cs[q * 6 + 5];
    C.dobj = rs[q * 4 + 3] + cs[q * 6 + 3] - cs[q * 6 + 4];
    C.gap = fabs(C.pobj - C.dobj);
    C.kkt = sqrt(omega * omega * C.errp * C.errp + C.errd * C.errd / (omega * omega) + C.gap * C.gap);
    C.abs_p = rs[8 + q * 3 + 0];
    C.abs_d = cs[12 + q * 2 + 0];
    C.abs_gap = C.gap;
    C.rel_p = C.abs_p / (1.0 + fmax(I.h_inf, fmax(rs[8 + q * 3 + 1], rs[8 + q * 3 + 2])));
    C.rel_d = C.abs_d / (1.0 + fmax(I.c_inf, cs[12 + q * 2 + 1]));
    C.rel_gap = C.gap / (1.0 + fmax(fabs(C.pobj), fabs(C.dobj)));
    C.r = sqrt(C.dxa2 / tau + C.dya2 / sigma);
    C.scale = sqrt(tau * b1sq + sigma * b2sq);
    C.rho = NAN;
    C.val_lo = 0.0;
    C.t_lo = 0.0;
    C.t_hi = 0.0;
    C.doublings = 0;
    C.bracketed = 0;
    C.last_dist = -1.0;
    if (mode != kModeCheck || I.force_kkt) {
      C.phase = kPhaseOff;  // KKT_omega is the restart metric: no bisection
    } else if (!(C.r > 0.0) || !isfinite(C.r)) {
      C.phase = kPhaseDone;  // invalid radius: numerical issue
    } else if (C.scale == 0.0) {
      C.phase = kPhaseDone;
      C.rho = 0.0;
    } else {
      C.phase = kPhaseExp;
      C.t_base = C.r / C.scale;
    }
  }
  if (nc < 2) I.cand[1].phase = kPhaseOff;
  if (mode == kModeCheck) I.pending = 0;
}

__global__ __launch_bounds__(kBlock) void k_cand_fin(Ranges rc, const double* __restrict__ rec_c,
                                                     Ranges rr, const double* __restrict__ rec_r,
                                                     Inst* __restrict__ inst, int mode) {
  cand_fin(blockIdx.x, rc, rec_c, rr, rec_r, inst, mode);
}

__device__ __forceinline__ double probe_t(const CandState& C, int p) {
  if (C.phase == kPhaseExp) return C.t_base * (double)(1u << p);
  return C.t_lo + (C.t_hi - C.t_lo) * (double)(p + 1) / (double)(kProbes + 1);
}

// One multisection pass: for the candidate blockIdx.y (if still searching) and
// every probe t, sum ||x(t) - x||^2 / tau and b1^T (x(t) - x) over the columns
// (eq. compute_zt_2).  Records: [candidate][workgroup][probe][2].
constexpr int kProbeNV = kProbes * 2;
template <typename T>
__device__ __forceinline__ void probe_cols_body(int b, int q, const Ranges& R, const T* x0, const T* x1,
                                                const double* g0, const double* g1, const DataPtrs<double>& d,
                                                const Inst* inst, int prec, double* rec, double* lds) {
  const Inst& I = inst[R.blk_inst[b]];
  if (I.status != kActive || I.check_due == 0 || I.precision != prec) return;
  const CandState& C = I.cand[q];
  if (C.phase != kPhaseExp && C.phase != kPhaseBisect) return;
  const double tau = I.eta_hat / I.omega;
  double tq[kProbes];
#pragma unroll
  for (int p = 0; p < kProbes; ++p) tq[p] = probe_t(C, p) * tau;
  double acc[kProbeNV];
#pragma unroll
  for (int i = 0; i < kProbeNV; ++i) acc[i] = 0.0;
  const double inv_tau = 1.0 / tau;
  const T* xs = q == 0 ? x0 : x1;
  const double* gs = q == 0 ? g0 : g1;
  const int j1 = R.blk_end[b];
  for (int j = R.blk_start[b] + (int)threadIdx.x; j < j1; j += kBlock) {
    const double lo = d.l[j], hi = d.u[j];
    const double xc = (double)xs[j];
    const double b1 = gs[j] - d.c[j];
#pragma unroll
    for (int p = 0; p < kProbes; ++p) {
      const double dx = clampd(xc + tq[p] * b1, lo, hi) - xc;
      acc[p * 2 + 0] += dx * dx * inv_tau;
      acc[p * 2 + 1] += b1 * dx;
    }
  }
  block_sum32_store(acc, lds, rec + ((size_t)q * R.nblk + b) * kProbeNV);
}

template <typename T>
__device__ __forceinline__ void probe_rows_body(int b, int q, const Ranges& R, const T* y0, const T* y1,
                                                const double* g0, const double* g1, const DataPtrs<double>& d,
                                                const double* D1, const Inst* inst, int prec, double* rec, double* lds) {
  const Inst& I = inst[R.blk_inst[b]];
  if (I.status != kActive || I.check_due == 0 || I.precision != prec) return;
  const CandState& C = I.cand[q];
  if (C.phase != kPhaseExp && C.phase != kPhaseBisect) return;
  const double sigma = I.eta_hat * I.omega;
  const int mz_end = I.row0 + I.m_zero;
  const double inv_sigma = 1.0 / sigma;
  const T* ys = q == 0 ? y0 : y1;
  const double* gs = q == 0 ? g0 : g1;
  // cone blocks first: y(t) = Proj onto diag(1/D1) (dual cone) of
  // y + t sigma b2, one task per block and probe (one inlined projection of a
  // kind); each wave's sums go to its own LDS slots.  (Done
  // before the element loop below, whose 48 per-probe values are then not
  // live across the projection: the kernel keeps more waves per SIMD.)
  __shared__ double cone_acc[kWavesPerBlock][kProbeNV];
  const bool cones = R.blk_soc0 && R.blk_soc1[b] > R.blk_soc0[b];
  const int wave = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
  if (cones) {
    for (int i = lane; i < kProbeNV; i += kWave) cone_acc[wave][i] = 0.0;
    wave_lds_order();
    double ld = 0.0, lb = 0.0;  // a lane's own blocks, all at probe lane % kProbes
    for_cone_tasks<kProbes>(R, b, [&](auto who, int r0, int dim, int kind, int p) {
      const double tp = probe_t(C, p) * sigma;
      double dd = 0.0, bd = 0.0;
      proj_cone(
          who, kind, true, dim, [&](int i) { return (double)ys[r0 + i] + tp * (d.h[r0 + i] - gs[r0 + i]); },
          [&](int i) { return 1.0 / D1[r0 + i]; },
          [&](int i, double pv) {
            const double yc = (double)ys[r0 + i];
            const double dy = pv - yc;
            dd += dy * dy;
            bd += (d.h[r0 + i] - gs[r0 + i]) * dy;
          });
      if constexpr (std::is_same_v<decltype(who), LaneTask>) {
        ld += dd;
        lb += bd;
      } else {
        dd = wave_sum(dd);
        bd = wave_sum(bd);
        if (lane == 0) {
          cone_acc[wave][p * 2 + 0] += dd * inv_sigma;
          cone_acc[wave][p * 2 + 1] += bd;
        }
      }
    });
#pragma unroll
    for (int off = kProbes; off < kWave; off <<= 1) {
      ld += __shfl_xor(ld, off);
      lb += __shfl_xor(lb, off);
    }
    wave_lds_order();
    if (lane < kProbes) {
      cone_acc[wave][lane * 2 + 0] += ld * inv_sigma;
      cone_acc[wave][lane * 2 + 1] += lb;
    }
    wave_lds_order();
  }
  double tq[kProbes];
#pragma unroll
  for (int p = 0; p < kProbes; ++p) tq[p] = probe_t(C, p) * sigma;
  double acc[kProbeNV];
#pragma unroll
  for (int i = 0; i < kProbeNV; ++i) acc[i] = 0.0;
  const int i1 = R.blk_end[b];
  for (int i = R.blk_start[b] + (int)threadIdx.x; i < i1; i += kBlock) {
    if (i >= I.soc_start) continue;  // cone block rows: above
    const bool zero_row = i < mz_end;
    const double yc = (double)ys[i];
    const double b2 = d.h[i] - gs[i];
#pragma unroll
    for (int p = 0; p < kProbes; ++p) {
      const double v = yc + tq[p] * b2;
      const double dy = (zero_row ? v : fmax(v, 0.0)) - yc;
      acc[p * 2 + 0] += dy * dy * inv_sigma;
      acc[p * 2 + 1] += b2 * dy;
    }
  }
  if (cones && lane == 0) {  // the wave's cone sums join acc in its lane 0
#pragma unroll
    for (int i = 0; i < kProbeNV; ++i) acc[i] += cone_acc[wave][i];
  }
  block_sum32_store(acc, lds, rec + ((size_t)q * R.nblk + b) * kProbeNV);
}

// A multisection pass, blockIdx.y the candidate: workgroups [0, rr.nblk) take the
// rows (cone blocks take longest, so they go first), the others the columns.
// (m = 2e4, n = 4e4: a launch each and the update, 8.7 + 8.7 + 12.2 us a pass; 7.6 +
// 4.5 here.  n = 5e5, m = 2e5: 15.6 + 11.0 + 24.4, and 21.7 + 10.3.)
template <typename T>
__global__ __launch_bounds__(kBlock) void k_probe(Ranges rc, Ranges rr, const T* __restrict__ x0,
                                                  const T* __restrict__ x1, const T* __restrict__ y0,
                                                  const T* __restrict__ y1, const double* __restrict__ gc0,
                                                  const double* __restrict__ gc1, const double* __restrict__ gr0,
                                                  const double* __restrict__ gr1, DataPtrs<double> d,
                                                  const double* __restrict__ D1, const Inst* __restrict__ inst, int prec,
                                                  double* __restrict__ rec_c, double* __restrict__ rec_r) {
  __shared__ double lds[kWavesPerBlock * kProbeNV];
  const int b = blockIdx.x;
  if (b < rr.nblk) probe_rows_body<T>(b, blockIdx.y, rr, y0, y1, gr0, gr1, d, D1, inst, prec, rec_r, lds);
  else probe_cols_body<T>(b - rr.nblk, blockIdx.y, rc, x0, x1, gc0, gc1, d, inst, prec, rec_c, lds);
}

__device__ __forceinline__ bool searching(const CandState& C) {
  return C.phase == kPhaseExp || C.phase == kPhaseBisect;
}

// A candidate's bracket from the sums of one multisection pass (Algorithm 3:
// exponential search from t0, then bisection; here kProbes points per pass);
// dist, val and tp in memory that may be indexed at run time.
__device__ __forceinline__ void probe_update(CandState& C, double eps, const double* dist, const double* val,
                                             const double* tp) {
  if (C.phase == kPhaseExp) {
    bool decided = false;
    for (int p = 0; p < kProbes; ++p) {
      const bool first = (C.doublings == 0 && p == 0);
      if (dist[p] > C.r) {
        if (first) {
          C.t_lo = 0.0;
          C.val_lo = 0.0;
        } else {
          C.t_lo = p > 0 ? tp[p - 1] : C.t_base * 0.5;
          // val_lo was recorded with the previous probe
        }
        C.t_hi = tp[p];
        C.phase = kPhaseBisect;
        decided = true;
        break;
      }
      if (!first && dist[p] <= C.last_dist) {  // saturated: z(2t) = z(t)
        C.phase = kPhaseDone;
        decided = true;
        break;
      }
      C.last_dist = dist[p];
      C.val_lo = val[p];
      C.t_lo = tp[p];
      C.doublings += 1;
    }
    if (!decided) {
      C.t_base = tp[kProbes - 1] * 2.0;
      if (C.doublings >= 64) C.phase = kPhaseDone;
    }
  } else {
    int last_in = -1;
    for (int p = 0; p < kProbes; ++p)
      if (dist[p] < C.r) last_in = p;
    const double new_hi = (last_in + 1 < kProbes) ? tp[last_in + 1] : C.t_hi;
    if (last_in >= 0) {
      C.t_lo = tp[last_in];
      C.val_lo = val[last_in];
    }
    C.t_hi = new_hi;
  }
  if (C.phase == kPhaseBisect && C.t_hi - C.t_lo <= eps * C.t_hi) C.phase = kPhaseDone;
}

// Work of a multisection pass that is one workgroup's: kBlock threads for each
// candidate q and each side (columns, rows), thread t of group 2 q + side.
constexpr int kProbeGroups = 2 * kMaxCand;
struct ProbeLds {
  double part[kProbeGroups][kBlock];     // partial sums of the groups
  double sums[kProbeGroups][kProbeNV];
  double dist[kMaxCand][kProbes], val[kMaxCand][kProbes], t[kMaxCand][kProbes];
};

// The brackets of both candidates from L.sums: first kProbes threads of a
// candidate's first group; C: its state.
__device__ __forceinline__ void probe_brackets(ProbeLds& L, int q, int p, CandState& C, double eps) {
  if (p < kProbes) {
    L.dist[q][p] = sqrt(L.sums[2 * q][p * 2] + L.sums[2 * q + 1][p * 2]);
    L.val[q][p] = L.sums[2 * q][p * 2 + 1] + L.sums[2 * q + 1][p * 2 + 1];
    L.t[q][p] = probe_t(C, p);
  }
  wave_lds_order();
  if (p == 0) probe_update(C, eps, L.dist[q], L.val[q], L.t[q]);
}

// Update every candidate's bracket from the records of one multisection pass.
// Thread t of a group adds value t % kProbeNV of every eighth record, eight loads
// in flight, and the group's partial sums are added in a fixed order.  (The four
// sums one after the other by 256 threads: 12.2 us at 40 + 20 records, 24.4 at
// 489 + 196; 4.5 and 10.3 here.)
__global__ __launch_bounds__(kProbeGroups* kBlock) void k_probe_fin(Ranges rc, const double* __restrict__ rec_c,
                                                                    Ranges rr, const double* __restrict__ rec_r,
                                                                    Inst* __restrict__ inst) {
  __shared__ ProbeLds L;
  const int iid = blockIdx.x;
  Inst& I = inst[iid];
  if (I.status != kActive || I.check_due == 0) return;
  if (!searching(I.cand[0]) && !searching(I.cand[1])) return;
  const int g = threadIdx.x / kBlock, t = threadIdx.x % kBlock, q = g >> 1;
  const bool rows = g & 1, on = searching(I.cand[q]);
  constexpr int R = kBlock / kProbeNV, U = 8;
  if (on) {
    const Ranges& side = rows ? rr : rc;
    const double* rec = (rows ? rec_r : rec_c) + (size_t)q * side.nblk * kProbeNV;
    const int i = t % kProbeNV, b1 = side.inst_blk0[iid + 1];
    int b = side.inst_blk0[iid] + t / kProbeNV;
    double acc = 0.0;
    for (; b + (U - 1) * R < b1; b += U * R) {
      double v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = rec[(size_t)(b + u * R) * kProbeNV + i];
#pragma unroll
      for (int u = 0; u < U; ++u) acc += v[u];
    }
    for (; b < b1; b += R) acc += rec[(size_t)b * kProbeNV + i];
    L.part[g][t] = acc;
  }
  __syncthreads();
  if (on && t < kProbeNV) {
    double s = L.part[g][t];
    for (int k = 1; k < R; ++k) s += L.part[g][k * kProbeNV + t];
    L.sums[g][t] = s;
  }
  __syncthreads();
  if (on && !rows && t < kWave) probe_brackets(L, q, t, I.cand[q], I.bisect_eps);
}

// Restart decision (Section 2.3), primal weight (Section 2.5), termination
// (Section 3) and the mixed-precision polish switch.  Thread 0 only.
__device__ __forceinline__ void check_decide(Inst& I) {
  if (I.status != kActive || I.check_due == 0) return;
  I.checks += 1;
  I.ray_due = 0;
  const int nc = I.use_avg ? 2 : 1;
  bool all_valid = true;
  for (int q = 0; q < nc; ++q) {
    CandState& C = I.cand[q];
    if (C.phase == kPhaseBisect) C.phase = kPhaseDone;  // pass budget spent: take t_lo
    if (C.phase == kPhaseExp) C.phase = kPhaseDone;
    if (I.force_kkt) C.rho = NAN;  // the gap is not computed
    else if (!(C.r > 0.0) || !isfinite(C.r)) C.rho = NAN;
    else if (C.scale == 0.0) C.rho = 0.0;
    else C.rho = C.val_lo / C.r;
    if (!(C.rho >= 0.0) || !isfinite(C.rho)) all_valid = false;
  }
  for (int q = 0; q < kMaxCand; ++q) {
    I.chk_rho[q] = q < nc ? I.cand[q].rho : NAN;
    I.chk_r[q] = q < nc ? I.cand[q].r : NAN;
  }
  if (I.has_anchor && !(I.rho_anchor >= 0.0 && isfinite(I.rho_anchor))) all_valid = false;
  if (I.has_prev && !(I.rho_prev >= 0.0 && isfinite(I.rho_prev))) all_valid = false;
  const bool use_kkt = I.force_kkt != 0 || !all_valid;
  int ch;
  if (I.method == 1) ch = 1;
  else if (I.method == 2 || nc == 1) ch = 0;
  else {
    const double m0 = use_kkt ? I.cand[0].kkt : I.cand[0].rho;
    const double m1 = use_kkt ? I.cand[1].kkt : I.cand[1].rho;
    ch = (m0 <= m1) ? 0 : 1;
  }
  CandState& C = I.cand[ch];
  const double mc = use_kkt ? C.kkt : C.rho;
  const double ma = use_kkt ? I.kkt_anchor : I.rho_anchor;
  const double mp = use_kkt ? I.kkt_prev : I.rho_prev;
  I.use_kkt = use_kkt;
  I.chosen = ch;
  I.pobj = C.pobj;
  I.dobj = C.dobj;
  I.abs_p = C.abs_p;
  I.abs_d = C.abs_d;
  I.abs_gap = C.abs_gap;
  I.rel_p = C.rel_p;
  I.rel_d = C.rel_d;
  I.rel_gap = C.rel_gap;
  const double amax = fmax(C.abs_p, fmax(C.abs_d, C.abs_gap));
  const double rmax = fmax(C.rel_p, fmax(C.rel_d, C.rel_gap));
  const bool optimal = (amax <= I.abs_tol) || (rmax <= I.rel_tol);
  bool restart = false;
  if ((double)I.k >= 0.223 * (double)I.kbar) restart = true;
  else if (I.has_anchor) {
    if (mc <= 0.4 * ma) restart = true;
    else if (I.has_prev && mc > mp && mc <= 0.8 * ma) restart = true;
  }
  I.optimal = optimal ? 1 : 0;
  I.switch_fp64 = 0;
  if (!optimal && I.precision == kFP32) {
    // Two signs that FP32 storage limits the attainable error.  Near the
    // tolerance (within 100x of rel_tol): stall_checks checks without a 10%
    // improvement of the best error (a slow linear descent still improves by
    // that much within the window; an error at a rounding floor does not).  At
    // any level: 8 x stall_checks checks without any new record low -- a
    // steady (even slow) descent keeps setting records, while an error that
    // fluctuates at a rounding floor sets them ever more rarely.
    if (!(rmax >= 0.9 * I.best_rel) || rmax > 100.0 * I.rel_tol) {
      I.best_rel = rmax;
      I.stall = 0;
    } else {
      I.stall += 1;
    }
    if (rmax < I.best_any) {
      I.best_any = rmax;
      I.stall_any = 0;
    } else {
      I.stall_any += 1;
    }
    if ((I.polish_tol > 0.0 && rmax <= I.polish_tol) ||
        (I.stall_checks > 0 && (I.stall >= I.stall_checks || I.stall_any >= 8 * I.stall_checks))) {
      I.switch_fp64 = 1;
      restart = true;
    }
  }
  if (optimal) {
    I.restart = 1;
    return;
  }
  if (isnan(rmax)) {
    I.restart = 0;
    I.status = kDone;
    I.exit_code = 8;
    return;
  }
  I.restart = restart ? 1 : 0;
  I.ray_due = I.infeas_on;
  if (restart) {
    const double dx = sqrt(C.dxa2), dy = sqrt(C.dya2);
    double w = I.omega;
    if (dx > 1e-10 && dy > 1e-10) w = exp(0.5 * log(dy / dx) + 0.5 * log(w));
    if (w > 1e5 || w < 1e-5) w = I.omega0;
    I.omega = w;
    I.rho_anchor = C.rho;
    I.kkt_anchor = sqrt(w * w * C.errp * C.errp + C.errd * C.errd / (w * w) + C.gap * C.gap);
    I.has_anchor = 1;
    I.has_prev = 0;
    I.k = 0;
    I.sum_eta = 0.0;
    I.t += 1;
    I.restarts += 1;
  } else {
    I.rho_prev = C.rho;
    I.kkt_prev = C.kkt;
    I.has_prev = 1;
  }
  // trial budget spent: stop after this check (k_check_end), once the
  // infeasibility tests of the check have run
  if (I.kbar >= I.max_iter) I.stop_max_iter = 1;
}

__global__ void k_decide(Inst* __restrict__ inst, int nb) {
  const int iid = blockIdx.x * blockDim.x + threadIdx.x;
  if (iid < nb) check_decide(inst[iid]);
}

// Apply a restart (anchor <- candidate, products refreshed from the FP64-value
// candidate products) or, for an optimal candidate, write the unscaled answer.
// Columns: x, G^T y, average sums, x_out = D2 x, lam_out = (c_hat - G^T y_hat)/D2.
template <typename T>
__device__ __forceinline__ void restart_cols(int b, const Ranges& R, const IterPtrs<T>& it, const IterPtrs<double>& it64,
                                             const double* g0, const double* g1,
                                             const DataPtrs<double>& d, const double* D2,
                                             double* xout, double* lamout,
                                             const Inst* inst, int prec) {
  const Inst& I = inst[R.blk_inst[b]];
  if (I.check_due == 0 || I.restart == 0 || I.precision != prec) return;
  const int ch = I.chosen;
  const T* xc = ch == 0 ? it.xh : it.xbar;
  const double* gc = ch == 0 ? g0 : g1;
  const int j1 = R.blk_end[b];
  for (int j = R.blk_start[b] + (int)threadIdx.x; j < j1; j += kBlock) {
    const double xv = (double)xc[j];
    const double gv = gc[j];
    if (I.optimal) {
      xout[j] = D2[j] * xv;
      lamout[j] = (d.c[j] - gv) / D2[j];
    } else if (I.switch_fp64) {
      it64.x[j] = xv;
      it64.xa[j] = xv;
      it64.xh[j] = xv;
      it64.gty[j] = gv;
      it64.gtya[j] = gv;
      it64.gtyh[j] = gv;
      it64.sx[j] = 0.0;
    } else {
      const T xt = (T)xv, gt = (T)gv;
      it.x[j] = xt;
      it.xa[j] = xt;
      it.gty[j] = gt;
      it.gtya[j] = gt;
      it.sx[j] = (T)0;
    }
  }
}

template <typename T>
__device__ __forceinline__ void restart_rows(int b, const Ranges& R, const IterPtrs<T>& it, const IterPtrs<double>& it64,
                                             const double* g0, const double* g1,
                                             const double* D1, double* yout,
                                             const Inst* inst, int prec) {
  const Inst& I = inst[R.blk_inst[b]];
  if (I.check_due == 0 || I.restart == 0 || I.precision != prec) return;
  const int ch = I.chosen;
  const T* yc = ch == 0 ? it.yh : it.ybar;
  const double* gc = ch == 0 ? g0 : g1;
  const int i1 = R.blk_end[b];
  for (int i = R.blk_start[b] + (int)threadIdx.x; i < i1; i += kBlock) {
    const double yv = (double)yc[i];
    const double gv = gc[i];
    if (I.optimal) {
      yout[i] = D1[i] * yv;
    } else if (I.switch_fp64) {
      it64.y[i] = yv;
      it64.ya[i] = yv;
      it64.yh[i] = yv;
      it64.gx[i] = gv;
      it64.gxa[i] = gv;
      it64.gxh[i] = gv;
      it64.sy[i] = 0.0;
    } else {
      const T yt = (T)yv, gt = (T)gv;
      it.y[i] = yt;
      it.ya[i] = yt;
      it.gx[i] = gt;
      it.gxa[i] = gt;
      it.sy[i] = (T)0;
    }
  }
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_restart(Ranges rc, Ranges rr, IterPtrs<T> it, IterPtrs<double> it64,
                                                    const double* __restrict__ gc0, const double* __restrict__ gc1,
                                                    const double* __restrict__ gr0, const double* __restrict__ gr1,
                                                    DataPtrs<double> d, const double* __restrict__ D1,
                                                    const double* __restrict__ D2, double* __restrict__ xout,
                                                    double* __restrict__ lamout, double* __restrict__ yout,
                                                    const Inst* __restrict__ inst, int prec) {
  const int b = blockIdx.x;
  if (b < rc.nblk) restart_cols<T>(b, rc, it, it64, gc0, gc1, d, D2, xout, lamout, inst, prec);
  else restart_rows<T>(b - rc.nblk, rr, it, it64, gr0, gr1, D1, yout, inst, prec);
}

__device__ __forceinline__ void check_end(Inst& I) {
  if (I.check_due == 0) return;
  if (I.optimal && I.status == kActive) {
    I.status = kDone;
    I.exit_code = 0;
  }
  if (I.stop_max_iter && I.status == kActive) {
    I.status = kDone;
    I.exit_code = 1;
  }
  if (I.switch_fp64 && I.status == kActive) {
    I.precision = kFP64;
    I.switch_fp64 = 0;
    I.best_rel = INFINITY;
    I.stall = 0;
    I.best_any = INFINITY;
    I.stall_any = 0;
  }
  I.check_due = 0;
  I.restart = 0;
  I.ray_due = 0;
}

__global__ void k_check_end(Inst* __restrict__ inst, int nb) {
  const int iid = blockIdx.x * blockDim.x + threadIdx.x;
  if (iid < nb) check_end(inst[iid]);
}

// ===========================================================================
// Infeasibility tests (option list of Section 3; exit codes 2-5)
// ===========================================================================
// The tests run on rays: the displacement of the PDHG output z_hat from the
// projected start point, r_x = Proj_rec(x_hat - x_start) onto the recession
// cone of the box and r_y = Proj_Kd(y_hat - y_start), in the rescaled space
// (both projections commute with the positive diagonal scaling).  Unscaled,
// G^T (D1 r_y) = D2^{-1} G_hat^T r_y and G (D2 r_x) = D1^{-1} G_hat r_x.
template <typename T>
__device__ __forceinline__ double ray_x(const T* xh, const double* xs0, const DataPtrs<double>& d, int j) {
  const double v = (double)xh[j] - xs0[j];
  const bool lf = isfinite(d.l[j]), uf = isfinite(d.u[j]);
  return lf && uf ? 0.0 : lf ? fmax(v, 0.0) : uf ? fmin(v, 0.0) : v;
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_ray_vec_cols(Ranges R, const T* __restrict__ xh,
                                                         const double* __restrict__ xs0, DataPtrs<double> d,
                                                         double* __restrict__ rx, const Inst* __restrict__ inst,
                                                         int prec) {
  const int b = blockIdx.x;
  const Inst& I = inst[R.blk_inst[b]];
  if (!mode_selects(I, kModeRay) || I.precision != prec) return;
  const int j1 = R.blk_end[b];
  for (int j = R.blk_start[b] + (int)threadIdx.x; j < j1; j += kBlock) rx[j] = ray_x(xh, xs0, d, j);
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_ray_vec_rows(Ranges R, const T* __restrict__ yh,
                                                         const double* __restrict__ ys0, const double* __restrict__ D1,
                                                         double* __restrict__ ry, const Inst* __restrict__ inst,
                                                         int prec) {
  const int b = blockIdx.x;
  const Inst& I = inst[R.blk_inst[b]];
  if (!mode_selects(I, kModeRay) || I.precision != prec) return;
  const int mz_end = I.row0 + I.m_zero;
  const int i1 = R.blk_end[b];
  for (int i = R.blk_start[b] + (int)threadIdx.x; i < i1; i += kBlock) {
    if (i >= I.soc_start) continue;  // cone block rows: below
    const double v = (double)yh[i] - ys0[i];
    ry[i] = i < mz_end ? v : fmax(v, 0.0);
  }
  // cone blocks: the unscaled ray D1 (y_hat - y_start) projected onto the dual cone,
  // stored scaled back by 1 / D1 like the other rows
  for_cone_blocks(R, b, [&](auto who, int r0, int dim, int kind) {
    proj_cone(
        who, kind, true, dim, [&](int i) { return D1[r0 + i] * ((double)yh[r0 + i] - ys0[r0 + i]); }, [](int) { return 1.0; },
        [&](int i, double p) { ry[r0 + i] = p / D1[r0 + i]; });
  });
}

// Where a check's rays go (rx null: every primal ray is 0).
struct RayOut {
  const double *xs0, *ys0;
  double *rx, *ry;
};

// All multisection passes of a restart check in one launch, one workgroup per
// instance of precision prec (the layouts that run trials in one workgroup per
// instance; no cone blocks there): the groups of k_probe_fin sum the whole
// instance with the arithmetic of k_probe and keep the candidates in LDS.  It is
// bound by each pass' chain of loads, exchanges and the bracket's update.
// (n = 500, m = 200: 7 passes of 14.8 us with one wave per candidate and side,
// its sums through memory; of 5.0 here.)  The decision and the rays of the check
// follow in the same launch.
template <typename T>
__global__ __launch_bounds__(kProbeGroups* kBlock) void k_probes_wg(const T* x0, const T* x1, const T* y0, const T* y1,
                                                                    const double* gc0, const double* gc1,
                                                                    const double* gr0, const double* gr1,
                                                                    DataPtrs<double> d, Inst* inst, int prec,
                                                                    int passes, RayOut ray) {
  __shared__ ProbeLds L;
  __shared__ CandState cand[kMaxCand];
  __shared__ double tq[kProbeGroups][kProbes];
  Inst& I = inst[blockIdx.x];
  if (I.status != kActive || I.check_due == 0 || I.precision != prec) return;  // uniform
  if (threadIdx.x < kMaxCand) cand[threadIdx.x] = I.cand[threadIdx.x];
  __syncthreads();
  const int g = threadIdx.x / kBlock, t = threadIdx.x % kBlock, q = g >> 1;
  const int lane = threadIdx.x & (kWave - 1), wave = t / kWave;
  const bool rows = g & 1;
  const double step = rows ? I.eta_hat * I.omega : I.eta_hat / I.omega, inv = 1.0 / step;
  const int mz_end = I.row0 + I.m_zero;
  for (int pass = 0; pass < passes; ++pass) {
    const bool on = searching(cand[q]);
    if (!searching(cand[0]) && !searching(cand[1])) break;  // uniform
    if (on && t < kProbes) tq[g][t] = probe_t(cand[q], t) * step;
    __syncthreads();
    if (on) {
      double acc[kProbeNV];
#pragma unroll
      for (int i = 0; i < kProbeNV; ++i) acc[i] = 0.0;
      if (!rows) {
        const T* xs = q == 0 ? x0 : x1;
        const double* gs = q == 0 ? gc0 : gc1;
        for (int j = I.col0 + t; j < I.col0 + I.cols; j += kBlock) {
          const double lo = d.l[j], hi = d.u[j];
          const double xc = (double)xs[j];
          const double b1 = gs[j] - d.c[j];
#pragma unroll
          for (int p = 0; p < kProbes; ++p) {
            const double dx = clampd(xc + tq[g][p] * b1, lo, hi) - xc;
            acc[p * 2 + 0] += dx * dx * inv;
            acc[p * 2 + 1] += b1 * dx;
            if (p % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // (16 probes' t at once would spill)
          }
        }
      } else {
        const T* ys = q == 0 ? y0 : y1;
        const double* gs = q == 0 ? gr0 : gr1;
        for (int i = I.row0 + t; i < I.row0 + I.rows; i += kBlock) {
          const bool zero_row = i < mz_end;
          const double yc = (double)ys[i];
          const double b2 = d.h[i] - gs[i];
#pragma unroll
          for (int p = 0; p < kProbes; ++p) {
            const double v = yc + tq[g][p] * b2;
            const double dy = (zero_row ? v : fmax(v, 0.0)) - yc;
            acc[p * 2 + 0] += dy * dy * inv;
            acc[p * 2 + 1] += b2 * dy;
            if (p % 4 == 3) __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
      const double s = wave_sum32(acc);
      if (lane < 32) L.part[g][wave * kProbeNV + (int)(__brev((unsigned)lane) >> 27)] = s;
    }
    __syncthreads();
    if (on && t < kProbeNV)
      L.sums[g][t] =
          ((L.part[g][t] + L.part[g][kProbeNV + t]) + L.part[g][2 * kProbeNV + t]) + L.part[g][3 * kProbeNV + t];
    __syncthreads();
    if (on && !rows && t < kWave) probe_brackets(L, q, t, cand[q], I.bisect_eps);
    __syncthreads();
  }
  if (threadIdx.x < kMaxCand) I.cand[threadIdx.x] = cand[threadIdx.x];
  __syncthreads();
  if (threadIdx.x == 0) check_decide(I);
  __syncthreads();
  if (!mode_selects(I, kModeRay)) return;
  for (int i = I.row0 + (int)threadIdx.x; i < I.row0 + I.rows; i += kProbeGroups * kBlock) {
    const double v = (double)y0[i] - ray.ys0[i];
    ray.ry[i] = i < mz_end ? v : fmax(v, 0.0);
  }
  if (ray.rx)
    for (int j = I.col0 + (int)threadIdx.x; j < I.col0 + I.cols; j += kProbeGroups * kBlock)
      ray.rx[j] = ray_x(x0, ray.xs0, d, j);
}
static_assert(kProbeNV == 32 && kWavesPerBlock == 4, "the sums of a pass are 32 values over four waves");

// Column terms, with lam = -(G_hat^T r_y)_j / D2_j (the unscaled -G^T r_y) and
// the unscaled bounds l_j = l_hat_j D2_j, u_j = u_hat_j D2_j:
//   [0] ||lam - Proj_Lambda lam||^2   [1] sum l lam+ - u lam- (finite bounds)
//   [2] its terms' magnitudes          [3] number of those terms
//   [4] c^T r_x (= c_hat^T r_x)         [5] its terms' magnitudes
constexpr int kRayColsNV = 6;
__device__ __forceinline__ void ray_cols(int b, const Ranges& R, const double* rx, const double* rgty,
                                         const DataPtrs<double>& d, const double* D2, const Inst* inst, double* rec) {
  __shared__ double lds[kWavesPerBlock * kRayColsNV];
  const Inst& I = inst[R.blk_inst[b]];
  if (!mode_selects(I, kModeRay)) return;
  double acc[kRayColsNV] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  const int j1 = R.blk_end[b];
  for (int j = R.blk_start[b] + (int)threadIdx.x; j < j1; j += kBlock) {
    const double dj = D2[j];
    const double lam = -rgty[j] / dj;
    const double lo = d.l[j], hi = d.u[j];
    const bool lf = isfinite(lo), uf = isfinite(hi);
    double viol;
    if (!lf && !uf) viol = lam;               // Lambda_j = {0}
    else if (!lf) viol = fmax(lam, 0.0);      // R-
    else if (!uf) viol = fmin(lam, 0.0);      // R+
    else viol = 0.0;                          // R
    acc[0] += viol * viol;
    if (lf) {
      const double t = (lo * dj) * fmax(lam, 0.0);
      acc[1] += t;
      acc[2] += fabs(t);
      acc[3] += 1.0;
    }
    if (uf) {
      const double t = -(hi * dj) * fmax(-lam, 0.0);
      acc[1] += t;
      acc[2] += fabs(t);
      acc[3] += 1.0;
    }
    const double cx = rx ? d.c[j] * rx[j] : 0.0;
    acc[4] += cx;
    acc[5] += fabs(cx);
  }
  block_sum_store<kRayColsNV>(acc, lds, rec + (size_t)b * kRayColsNV);
}

__global__ __launch_bounds__(kBlock) void k_ray_cols(Ranges R, const double* __restrict__ rx,
                                                     const double* __restrict__ rgty, DataPtrs<double> d,
                                                     const double* __restrict__ D2, const Inst* __restrict__ inst,
                                                     double* __restrict__ rec) {
  ray_cols(blockIdx.x, R, rx, rgty, d, D2, inst, rec);
}

// Row terms: [0] h^T r_y (= h_hat^T r_y), [1] its terms' magnitudes,
// [2] ||G r_x - Proj_Kd*(G r_x)||^2 with (G r_x)_i = (G_hat r_x)_i / D1_i
// (zero when no instance has a nonzero primal ray: rgx null).
constexpr int kRayRowsNV = 3;
template <bool CONES>
__device__ __forceinline__ void ray_rows(int b, const Ranges& R, const double* ry, const double* rgx,
                                         const DataPtrs<double>& d, const double* D1, const Inst* inst, double* rec) {
  __shared__ double lds[kWavesPerBlock * kRayRowsNV];
  const Inst& I = inst[R.blk_inst[b]];
  if (!mode_selects(I, kModeRay)) return;
  const int mz_end = I.row0 + I.m_zero;
  double acc[kRayRowsNV] = {0.0, 0.0, 0.0};
  const int i1 = R.blk_end[b];
  for (int i = R.blk_start[b] + (int)threadIdx.x; i < i1; i += kBlock) {
    const double t = d.h[i] * ry[i];
    acc[0] += t;
    acc[1] += fabs(t);
    if (rgx && i < I.soc_start) {
      const double r = rgx[i] / D1[i];
      const double res = i < mz_end ? r : fmin(r, 0.0);
      acc[2] += res * res;
    }
  }
  // cone blocks: the unscaled G r_x against the block's cone
  if (CONES && rgx)
    for_cone_blocks(R, b, [&](auto who, int r0, int dim, int kind) {
      proj_cone(
          who, kind, false, dim, [&](int i) { return rgx[r0 + i] / D1[r0 + i]; }, [](int) { return 1.0; },
          [&](int i, double p) {
            const double res = rgx[r0 + i] / D1[r0 + i] - p;
            acc[2] += res * res;
          });
    });
  block_sum_store<kRayRowsNV>(acc, lds, rec + (size_t)b * kRayRowsNV);
}

__global__ __launch_bounds__(kBlock) void k_ray_rows(Ranges R, const double* __restrict__ ry,
                                                     const double* __restrict__ rgx, DataPtrs<double> d,
                                                     const double* __restrict__ D1, const Inst* __restrict__ inst,
                                                     double* __restrict__ rec) {
  ray_rows<true>(blockIdx.x, R, ry, rgx, d, D1, inst, rec);
}

// gamma_N = N u / (1 - N u), u = 2^-53: relative error bound of a sum of N terms.
__device__ __forceinline__ double rounding_bound(double count) {
  const double nu = fmax(count, 1.0) * 0x1p-53;
  return nu / (1.0 - nu);
}

// Ratios, trend counters and the exit decision of the infeasibility tests.
// Priority: high-accuracy primal (3), high-accuracy dual (5), low-accuracy
// primal (2), low-accuracy dual (4); a tolerance of 0 never passes.
__device__ __forceinline__ void ray_fin(int iid, const Ranges& rc, const double* rec_c, const Ranges& rr,
                                        const double* rec_r, Inst* inst) {
  __shared__ double lds[kWavesPerBlock * kRayColsNV];
  Inst& I = inst[iid];
  if (!mode_selects(I, kModeRay)) return;
  double cs[kRayColsNV], rs[kRayRowsNV];
  reduce_records<kRayColsNV, kRayColsNV>(rec_c, rc.inst_blk0[iid], rc.inst_blk0[iid + 1], lds, cs);
  reduce_records<kRayRowsNV, kRayRowsNV>(rec_r, rr.inst_blk0[iid], rr.inst_blk0[iid + 1], lds, rs);
  if (threadIdx.x != 0) return;
  const double f = rs[0] + cs[1];
  const double fmag = rs[1] + cs[2];
  const double ratio_p = f > rounding_bound((double)I.rows + cs[3]) * fmag ? sqrt(cs[0]) / f : (double)INFINITY;
  const double g = -cs[4];
  const double ratio_d = g > rounding_bound((double)I.cols) * cs[5] ? sqrt(rs[2]) / g : (double)INFINITY;
  const double pobj = I.cand[0].pobj, dobj = I.cand[0].dobj;
  const bool up_p = I.has_prev_obj && dobj > I.prev_dobj;
  const bool up_d = I.has_prev_obj && -pobj > I.prev_negp;
  I.prev_dobj = dobj;
  I.prev_negp = -pobj;
  I.has_prev_obj = 1;
  I.trend_p = (ratio_p < I.eps_inf[0] && up_p) ? I.trend_p + 1 : 0;
  I.trend_d = (ratio_d < I.eps_inf[1] && up_d) ? I.trend_d + 1 : 0;
  I.ratio_p = ratio_p;
  I.ratio_d = ratio_d;
  int code = 0;
  if (ratio_p < I.eps_inf[2]) code = 3;
  else if (ratio_d < I.eps_inf[3]) code = 5;
  else if (I.trend_p >= kTrendChecks) code = 2;
  else if (I.trend_d >= kTrendChecks) code = 4;
  if (code) {
    I.status = kDone;
    I.exit_code = code;
    I.restart = 0;
    I.switch_fp64 = 0;
  }
}

__global__ __launch_bounds__(kBlock) void k_ray_fin(Ranges rc, const double* __restrict__ rec_c, Ranges rr,
                                                    const double* __restrict__ rec_r, Inst* __restrict__ inst) {
  ray_fin(blockIdx.x, rc, rec_c, rr, rec_r, inst);
}

// Device warm starts into the packed FP64 start vector.
template <typename TW>
__global__ void k_pack_warm(const void* const* __restrict__ src, const int32_t* __restrict__ off, int B,
                            double* __restrict__ out, int32_t* __restrict__ nan_flag) {
  for (int b = blockIdx.y; b < B; b += gridDim.y) {
    const int o0 = off[b], len = off[b + 1] - off[b];
    const TW* sp = static_cast<const TW*>(src[b]);
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < len; e += gridDim.x * blockDim.x) {
      const double v = sp ? (double)sp[e] : 0.0;
      if (isnan(v)) *nan_flag = 1;
      out[o0 + e] = v;
    }
  }
}

// Evaluated point (start point or final point): termination test and output.
__device__ __forceinline__ void eval_fin(Inst& I, int mode) {
  if (!mode_selects(I, mode)) return;
  const CandState& C = I.cand[0];
  I.pobj = C.pobj;
  I.dobj = C.dobj;
  I.abs_p = C.abs_p;
  I.abs_d = C.abs_d;
  I.abs_gap = C.abs_gap;
  I.rel_p = C.rel_p;
  I.rel_d = C.rel_d;
  I.rel_gap = C.rel_gap;
  if (mode == kModeEvalStart) {
    const double amax = fmax(C.abs_p, fmax(C.abs_d, C.abs_gap));
    const double rmax = fmax(C.rel_p, fmax(C.rel_d, C.rel_gap));
    I.optimal = ((amax <= I.abs_tol) || (rmax <= I.rel_tol)) ? 1 : 0;
  } else {
    I.optimal = 0;
  }
}

__global__ void k_eval_fin(Inst* __restrict__ inst, int nb, int mode) {
  const int iid = blockIdx.x * blockDim.x + threadIdx.x;
  if (iid < nb) eval_fin(inst[iid], mode);
}

// Write the evaluated point (x_hat, y_hat) unscaled.  Start mode: only for
// instances found optimal (which then stop); final mode: every selected instance.
template <typename T>
__device__ __forceinline__ void eval_out(int b, bool cols, const Ranges& R, const T* xh, const T* yh, const double* g0,
                                         const DataPtrs<double>& d, const double* D1, const double* D2, double* xout,
                                         double* lamout, double* yout, const Inst* inst, int prec, int mode) {
  const Inst& I = inst[R.blk_inst[b]];
  if (!mode_selects(I, mode) || I.precision != prec) return;
  if (mode == kModeEvalStart && !I.optimal) return;
  const int e = R.blk_end[b];
  if (cols) {
    for (int j = R.blk_start[b] + (int)threadIdx.x; j < e; j += kBlock) {
      xout[j] = D2[j] * (double)xh[j];
      lamout[j] = (d.c[j] - g0[j]) / D2[j];
    }
  } else {
    for (int i = R.blk_start[b] + (int)threadIdx.x; i < e; i += kBlock) yout[i] = D1[i] * (double)yh[i];
  }
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_eval_out(Ranges rc, Ranges rr, const T* __restrict__ xh,
                                                     const T* __restrict__ yh, const double* __restrict__ g0,
                                                     DataPtrs<double> d, const double* __restrict__ D1,
                                                     const double* __restrict__ D2, double* __restrict__ xout,
                                                     double* __restrict__ lamout, double* __restrict__ yout,
                                                     const Inst* __restrict__ inst, int prec, int mode) {
  const bool cols = (int)blockIdx.x < rc.nblk;
  eval_out<T>(cols ? (int)blockIdx.x : (int)blockIdx.x - rc.nblk, cols, cols ? rc : rr, xh, yh, g0, d, D1, D2, xout,
              lamout, yout, inst, prec, mode);
}

__device__ __forceinline__ void eval_start_end(Inst& I) {
  if (I.status == kActive && I.optimal) {
    I.status = kDone;
    I.exit_code = 0;
  }
}

__global__ void k_eval_start_end(Inst* __restrict__ inst, int nb) {
  const int iid = blockIdx.x * blockDim.x + threadIdx.x;
  if (iid < nb) eval_start_end(inst[iid]);
}

// Counts of active instances per precision, for the host loop.
__global__ void k_summary(const Inst* __restrict__ inst, int nb, int32_t* __restrict__ out) {
  __shared__ int32_t cnt[2];
  if (threadIdx.x < 2) cnt[threadIdx.x] = 0;
  __syncthreads();
  int a32 = 0, a64 = 0;
  for (int i = threadIdx.x; i < nb; i += blockDim.x) {
    if (inst[i].status == kActive) {
      if (inst[i].precision == kFP32) ++a32;
      else ++a64;
    }
  }
  atomicAdd(&cnt[0], a32);
  atomicAdd(&cnt[1], a64);
  __syncthreads();
  if (threadIdx.x == 0) {
    out[0] = cnt[0];
    out[1] = cnt[1];
  }
}

__global__ void k_timeout(Inst* __restrict__ inst, int nb) {
  const int iid = blockIdx.x * blockDim.x + threadIdx.x;
  if (iid >= nb) return;
  if (inst[iid].status == kActive) {
    inst[iid].status = kDone;
    inst[iid].exit_code = 6;
  }
}

// Apply a pending Halpern commit (used to export the internal state at exit).
template <typename T>
__global__ __launch_bounds__(kBlock) void k_flush_commit(Ranges R, T* __restrict__ z,
                                                         const T* __restrict__ zh, const T* __restrict__ za,
                                                         T* __restrict__ g, const T* __restrict__ gh,
                                                         const T* __restrict__ ga, T* __restrict__ s,
                                                         const Inst* __restrict__ inst, int prec) {
  const int b = blockIdx.x;
  const Inst& I = inst[R.blk_inst[b]];
  if (I.pending == 0 || I.precision != prec) return;
  const double ca = I.ca, cb = I.cb, beta = I.beta, etak = I.eta_k;
  const bool avg = I.use_avg != 0;
  const int j1 = R.blk_end[b];
  for (int j = R.blk_start[b] + (int)threadIdx.x; j < j1; j += kBlock) {
    const double zhv = (double)zh[j];
    z[j] = (T)(ca * ((1.0 + beta) * zhv - beta * (double)z[j]) + cb * (double)za[j]);
    g[j] = (T)(ca * ((1.0 + beta) * (double)gh[j] - beta * (double)g[j]) + cb * (double)ga[j]);
    if (avg) s[j] = (T)((double)s[j] + etak * zhv);
  }
}

__global__ void k_clear_pending(Inst* __restrict__ inst, int nb) {
  const int iid = blockIdx.x * blockDim.x + threadIdx.x;
  if (iid < nb) inst[iid].pending = 0;
}

// ===========================================================================
// Set-up: diagonal rescaling (Section 2.6), norms, start point
// ===========================================================================

constexpr int kScaleLdsThreads = 1024;

// The scaling passes work on both sides at once: each computes, from the D1 and D2
// of the pass before, every row's and every column's statistic -- max |D1_i a_ij D2_j|
// (Ruiz, kScaleMax) or the sum of its squares (the 2-norm pass, kScaleSquares) --
// and from it the new factor.  A statistic of 0, or beyond FP64's range, keeps the factor.
enum { kScaleMax = 0, kScaleSquares = 1 };
__device__ __forceinline__ double scaled_factor(double D, double stat, int mode) {
  if (!(stat > 0.0) || !(stat <= __DBL_MAX__)) return D;
  return D / (mode == kScaleMax ? sqrt(stat) : sqrt(sqrt(stat)));
}

// One side of the matrix in row blocks: rows of G (own factor D1, the gathered one
// D2) or columns (own D2, gathered D1).  An entry's scaled value is
// (D1_i a_ij) D2_j on either side.
struct ScaleSide {
  RowBlocks rb;
  const int32_t *ptr, *idx;
  const double* val;
  const double *own, *other;  // null: all ones
  int cols;
  __device__ __forceinline__ double entry(double o, double a, double g) const {
    return cols ? (g * a) * o : (o * a) * g;
  }
};

// Row block b of a side: the entries' values and gathered factors in LDS (a block of
// several rows), then fn(row, own factor, first entry, end, lanes of the row, this
// lane) per row, entries relative to the block; for a single row of any length,
// fn1(row, own factor).  Latency bound like the trial products, and as they are
// done: all indices, then all gathers in flight.
template <class Fn, class Fn1>
__device__ __forceinline__ void scale_block(const ScaleSide& S, int b, double (*lds)[kRowBlockCap], const Fn& fn,
                                            const Fn1& fn1) {
  const int r0 = S.rb.blk_row0[b], r1 = S.rb.blk_row1[b], R = r1 - r0;
  const int q0 = S.ptr[r0], n = S.ptr[r1] - q0;
  const int tid = threadIdx.x;
  if (R == 1) {
    fn1(r0, S.own ? S.own[r0] : 1.0);
    return;
  }
  for (int i0 = 0; i0 < n; i0 += 4 * kBlock) {
    int c[4];
    double v[4], g[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = q0 + min(i0 + u * kBlock + tid, n - 1);
      c[u] = S.idx[i];
      v[u] = S.val[i];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) g[u] = S.other ? S.other[c[u]] : 1.0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      lds[0][i0 + u * kBlock + tid] = v[u];
      lds[1][i0 + u * kBlock + tid] = g[u];
    }
  }
  __syncthreads();
  int T = kWave;
  while (T > 1 && T * R > kBlock) T >>= 1;
  for (int g = tid / T; g < (R + kBlock / T - 1) / (kBlock / T) * (kBlock / T); g += kBlock / T) {
    const int r = r0 + min(g, R - 1);
    fn(r, S.own ? S.own[r] : 1.0, S.ptr[r] - q0, S.ptr[r + 1] - q0, T, tid & (T - 1), g < R);
  }
}

// One scaling pass over row blocks: workgroups [0, a.rb.nblk) take the rows, the
// others the columns.  (m = 2e4, n = 4e4, nnz = 3e5: a launch of 8.7 us where the two
// statistics and the two updates were four of 18 + 18 + 4.6 + 4.6 us.)
__global__ __launch_bounds__(kBlock) void k_scale_pass(ScaleSide a, ScaleSide c, int mode, double* __restrict__ D1o,
                                                       double* __restrict__ D2o) {
  __shared__ double lds[2][kRowBlockCap];
  __shared__ double red[kWavesPerBlock];
  const bool cols = (int)blockIdx.x >= a.rb.nblk;
  const ScaleSide& S = cols ? c : a;
  double* out = cols ? D2o : D1o;
  const int b = (int)blockIdx.x - (cols ? a.rb.nblk : 0);
  scale_block(
      S, b, lds,
      [&](int r, double own, int i0, int i1, int T, int li, bool live) {
        double s = 0.0;
        for (int i = i0 + li; i < i1; i += T) {
          if (mode == kScaleMax) {
            s = fmax(s, S.entry(own, fabs(lds[0][i]), lds[1][i]));
          } else {
            const double e = S.entry(own, lds[0][i], lds[1][i]);
            s += e * e;
          }
        }
        for (int off = T >> 1; off > 0; off >>= 1) {
          const double o = __shfl_xor(s, off, kWave);
          s = mode == kScaleMax ? fmax(s, o) : s + o;
        }
        if (li == 0 && live) out[r] = scaled_factor(own, s, mode);
      },
      [&](int r, double own) {
        double s = 0.0;
        for (int q = S.ptr[r] + (int)threadIdx.x; q < S.ptr[r + 1]; q += kBlock) {
          const double g = S.other ? S.other[S.idx[q]] : 1.0;
          if (mode == kScaleMax) {
            s = fmax(s, S.entry(own, fabs(S.val[q]), g));
          } else {
            const double e = S.entry(own, S.val[q], g);
            s += e * e;
          }
        }
        s = mode == kScaleMax ? wave_max(s) : wave_sum(s);
        if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = s;
        __syncthreads();
        if (threadIdx.x == 0) {
          s = red[0];
          for (int w = 1; w < kWavesPerBlock; ++w) s = mode == kScaleMax ? fmax(s, red[w]) : s + red[w];
          out[r] = scaled_factor(own, s, mode);
        }
      });
}

// All scaling passes and the scaled values of an instance by one workgroup, its
// matrix (both sides) and the factors of two passes in LDS, a thread per row or
// column: an instance that k_trials_lds takes with short rows (this needs 24 bytes
// per nonzero and 20 per row and column, fewer than that kernel in FP64).  Each pass
// is bound by its longest row's chain of LDS reads.  rec: the instance's largest
// magnitude at its first row block, 0 at its others.  (n = 500, m = 200, 2500
// nonzeros: 11 launches of 5.4 us and the values' 5.7 before, 33 here.)
__global__ __launch_bounds__(kScaleLdsThreads) void k_scale_lds(MatPtrs<double> A, MatPtrs<double> AT,
                                                                const int32_t* __restrict__ iblk, int passes, int ruiz,
                                                                double* __restrict__ D1, double* __restrict__ D2,
                                                                double* __restrict__ v64, float* __restrict__ v32,
                                                                double* __restrict__ vt64, float* __restrict__ vt32,
                                                                const Inst* __restrict__ inst, double* __restrict__ rec) {
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];
  __shared__ double red[kScaleLdsThreads / kWave];
  const int iid = blockIdx.x, tid = threadIdx.x;
  const Inst& I = inst[iid];
  const int r0 = I.row0, m = I.rows, c0 = I.col0, n = I.cols;
  const int q0 = A.ptr[r0], nnz = A.ptr[r0 + m] - q0;
  const int t0 = AT.ptr[c0];
  double* va = reinterpret_cast<double*>(dyn);
  double* vt = va + nnz;
  double* d = vt + nnz;  // factors: rows and columns of one pass, then of the other
  int32_t* ci = reinterpret_cast<int32_t*>(d + 2 * (m + n));
  int32_t* ri = ci + nnz;
  int32_t* ptr = ri + nnz;  // first entries of the rows, then of the columns
  for (int i = tid; i < nnz; i += kScaleLdsThreads) {
    va[i] = A.val[q0 + i];
    vt[i] = AT.val[t0 + i];
    ci[i] = m + A.idx[q0 + i] - c0;  // places in d
    ri[i] = AT.idx[t0 + i] - r0;
  }
  for (int i = tid; i < m + n; i += kScaleLdsThreads) {
    d[i] = 1.0;
    ptr[i] = i < m ? A.ptr[r0 + i] - q0 : AT.ptr[c0 + i - m] - t0;
  }
  __syncthreads();
  const auto bounds = [&](int i, int& b, int& e) {  // entries of row i, or column i - m
    b = ptr[i];
    e = i == m - 1 || i == m + n - 1 ? nnz : ptr[i + 1];
  };
  const double* from = d;
  double* to = d + (m + n);
  for (int pass = 0; pass < passes; ++pass) {
    const int mode = pass < ruiz ? kScaleMax : kScaleSquares;
    for (int i = tid; i < m + n; i += kScaleLdsThreads) {
      const bool row = i < m;
      const double* v = row ? va : vt;
      const int32_t* at = row ? ci : ri;
      const double own = from[i];
      int b, e;
      bounds(i, b, e);
      double s = 0.0;
      for (; b < e; b += 4) {
        double a[4], g[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int k = min(b + u, e - 1);
          a[u] = v[k];
          g[u] = from[at[k]];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const double x = row ? (own * a[u]) * g[u] : (g[u] * a[u]) * own;
          if (mode == kScaleMax) s = fmax(s, fabs(x));
          else if (b + u < e) s += x * x;
        }
      }
      to[i] = scaled_factor(own, s, mode);
    }
    __syncthreads();
    const double* t = from;
    from = to;
    to = const_cast<double*>(t);
  }
  double big = 0.0;
  for (int i = tid; i < m + n; i += kScaleLdsThreads) {
    const bool row = i < m;
    const double own = from[i];
    (row ? D1 + r0 : D2 + c0 - m)[i] = own;
    int b, e;
    bounds(i, b, e);
    for (; b < e; ++b) {
      const double x = row ? (own * va[b]) * from[ci[b]] : (from[ri[b]] * vt[b]) * own;
      (row ? v64 + q0 : vt64 + t0)[b] = x;
      (row ? v32 + q0 : vt32 + t0)[b] = (float)x;
      big = fmax(big, fabs(x));
    }
  }
  big = wave_max(big);
  if ((tid & (kWave - 1)) == 0) red[tid / kWave] = big;
  __syncthreads();
  for (int b = iblk[iid] + tid; b < iblk[iid + 1]; b += kScaleLdsThreads) {
    double x = 0.0;
    if (b == iblk[iid])
      for (int w = 0; w < kScaleLdsThreads / kWave; ++w) x = fmax(x, red[w]);
    rec[b] = x;
  }
}

// Scaled values of both sides in FP64 and FP32, and per row block of G the largest
// magnitude (rec, may be null).
__global__ __launch_bounds__(kBlock) void k_scale_values(ScaleSide a, ScaleSide c, double* __restrict__ v64,
                                                         float* __restrict__ v32, double* __restrict__ vt64,
                                                         float* __restrict__ vt32, double* __restrict__ rec) {
  __shared__ double lds[2][kRowBlockCap];
  __shared__ double red[kWavesPerBlock];
  const bool cols = (int)blockIdx.x >= a.rb.nblk;
  const ScaleSide& S = cols ? c : a;
  double* o64 = cols ? vt64 : v64;
  float* o32 = cols ? vt32 : v32;
  const int b = (int)blockIdx.x - (cols ? a.rb.nblk : 0);
  double big[1] = {0.0};
  scale_block(
      S, b, lds,
      [&](int, double own, int i0, int i1, int T, int li, bool live) {
        if (!live) return;
        for (int i = i0 + li; i < i1; i += T) {  // (each entry read and written by one lane)
          const double e = S.entry(own, lds[0][i], lds[1][i]);
          lds[0][i] = e;
          big[0] = fmax(big[0], fabs(e));
        }
      },
      [&](int r, double own) {
        for (int q = S.ptr[r] + (int)threadIdx.x; q < S.ptr[r + 1]; q += kBlock) {
          const double e = S.entry(own, S.val[q], S.other ? S.other[S.idx[q]] : 1.0);
          o64[q] = e;
          o32[q] = (float)e;
          big[0] = fmax(big[0], fabs(e));
        }
      });
  const int r0 = S.rb.blk_row0[b], r1 = S.rb.blk_row1[b];
  __syncthreads();
  if (r1 - r0 > 1) {
    const int q0 = S.ptr[r0], n = S.ptr[r1] - q0;
    for (int i = threadIdx.x; i < n; i += kBlock) {
      o64[q0 + i] = lds[0][i];
      o32[q0 + i] = (float)lds[0][i];
    }
  }
  if (!cols && rec) block_summax_store<1, 0>(big, red, rec + b);
}

// The same passes on band tiles (problems that take them): the statistics by the
// band kernel's sweep over the unscaled values in entry order, one launch for both
// matrices, without their own factor, which the update applies to the windows'
// results.  (Gathers from an L2 window instead of the whole vector: m = 2.5e5,
// n = 5e5, nnz = 1.35e7: 157 us per side of a pass from the CSR, 138 us here for
// both sides; m = 2e5, n = 5e5, nnz = 5e6: 49 per side, 63 here for both.)
template <class OP>
__global__ __launch_bounds__(kWave) void k_scale_bands(BandTiles b1, const double* __restrict__ v1,
                                                                    const double* __restrict__ D2,
                                                                    double* __restrict__ part1, int64_t M, BandTiles b2,
                                                                    const double* __restrict__ v2,
                                                                    const double* __restrict__ D1,
                                                                    double* __restrict__ part2, int64_t N) {
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];
  const bool second = (int)blockIdx.x >= b1.nslot;
  const BandTiles& bt = second ? b2 : b1;
  const BandTile t = bt.slot[(int)blockIdx.x - (second ? b1.nslot : 0)];
  double* acc = reinterpret_cast<double*>(dyn);
  band_tile_product<double, double, double, OP>(bt, t, acc, second ? v2 : v1, second ? D1 : D2, [] { return false; },
                                                PutPart<double>(t, second ? part2 : part1, second ? N : M));
}

// D1 (elements [0, M)) and D2 (the next N) from the windows' statistics, which lack the
// element's own factor d: |a| D_other at most, or the sum of (a D_other)^2, where the
// statistic proper is d times the one and d^2 times the other.  Once the Ruiz passes have
// made d about 1 / (a D_other), the squares without it leave FP64's range for rows of
// magnitude beyond 1e154 or below 1e-154, whose scaled entries are about 1 all the same
// (row_scale 1e-157: d^2 infinite, the factor 0).  So whatever is not well inside
// the range is taken again from the element's entries, as the row blocks take it; what
// lies inside lost at most 2^-1043 of a sum of 2^-900.
__global__ void k_scale_bands_update(ScaleSide a, ScaleSide c, const double* __restrict__ part1, int P1, int64_t M,
                                     const double* __restrict__ part2, int P2, int64_t N, int mode,
                                     double* __restrict__ D1o, double* __restrict__ D2o) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool live = e < M + N, second = e >= M;
  const int i = (int)(second ? e - M : e);
  const auto inside = [](double v) { return v >= 0x1p-900 && v <= 0x1p900; };
  double d = 1.0, stat = 0.0;
  int q0 = 0, q1 = 0;  // entries to be taken again
  if (live) {
    const int64_t n = second ? N : M;
    const double* part = second ? part2 : part1;
    const int P = second ? P2 : P1;
    double s = part[i];
    for (int p = 1; p < P; ++p) s = mode == kScaleMax ? fmax(s, part[(size_t)p * n + i]) : s + part[(size_t)p * n + i];
    d = (second ? c : a).own[i];
    const double f = mode == kScaleMax ? d : d * d;
    stat = f * s;
    if (!inside(s) || !inside(f) || !inside(stat)) {  // (an empty row has none, and its statistic is 0)
      q0 = (second ? c : a).ptr[i];
      q1 = (second ? c : a).ptr[i + 1];
    }
  }
  const int lane = threadIdx.x & (kWave - 1);
#pragma unroll 1
  for (unsigned long long left = __ballot(q1 > q0); left; left &= left - 1) {  // by the whole wave
    const int from = __ffsll(left) - 1;
    const int end = __shfl(q1, from);
    const ScaleSide& S = __shfl((int)second, from) ? c : a;
    const double own = __shfl(d, from);
    double s = 0.0;
    for (int q = __shfl(q0, from) + lane; q < end; q += kWave) {
      const double x = S.entry(own, S.val[q], S.other[S.idx[q]]);
      s = mode == kScaleMax ? fmax(s, fabs(x)) : s + x * x;
    }
    s = mode == kScaleMax ? wave_max(s) : wave_sum(s);
    if (lane == from) stat = s;
  }
  if (live) (second ? D2o : D1o)[i] = scaled_factor(d, stat, mode);
}

// Scaled band-entry values from the unscaled ones (in place where src == v64), and
// per band-tile the largest magnitude.  A tile's own factors sit in LDS by slot.
__device__ __forceinline__ void band_scale_tile(const BandTiles& bt, const BandTile& t, bool cols, double* own,
                                                const double* __restrict__ D_own, const double* __restrict__ D_other,
                                                const double* src, double* v64, float* __restrict__ v32,
                                                double* __restrict__ rec) {
  const int lane = threadIdx.x & (kWave - 1);
  for (int i = lane; i < t.nrows; i += kWave) {
    const double o = D_own[t.row0 + i];
    own[i] = o;
  }
  for (int i = lane; i < t.nfold; i += kWave) {
    const uint2 f = bt.fold[t.fold0 + i];
    const double o = D_own[t.row0 + (int)(f.x & 0xFFFFu)];
    for (uint32_t q = f.y; q < f.y + (f.x >> 16); ++q) own[q] = o;
  }
  if (lane == 0) own[bt.slots - 1] = 0.0;  // the padding's sink (its values are 0)
  wave_lds_order();
  const double* other = D_other + t.col0;
  double big = 0.0;
  constexpr int U = 8;  // the padding makes whole groups of kBandUnroll
  const int end = t.start + t.nit * kBandUnroll * kWave;
  for (int e0 = t.start + lane; e0 < end; e0 += U * kWave) {
    uint32_t pk[U];
    double v[U], g[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      pk[u] = bt.pk[e0 + u * kWave];
      v[u] = src[e0 + u * kWave];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) g[u] = other[pk[u] >> kBandSlotBits];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const double o = own[pk[u] & ((1u << kBandSlotBits) - 1u)];
      const double e = cols ? (g[u] * v[u]) * o : (o * v[u]) * g[u];
      v64[e0 + u * kWave] = e;
      v32[e0 + u * kWave] = (float)e;
      big = fmax(big, fabs(e));
    }
  }
  big = wave_max(big);
  if (rec && lane == 0 && t.tile >= 0) rec[t.tile] = big;
}

__global__ __launch_bounds__(kWave) void k_scale_bands_values(BandTiles b1, const double* s1, double* v1,
                                                                           float* __restrict__ f1, BandTiles b2,
                                                                           const double* s2, double* v2,
                                                                           float* __restrict__ f2,
                                                                           const double* __restrict__ D1,
                                                                           const double* __restrict__ D2,
                                                                           double* __restrict__ rec) {
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];
  const bool second = (int)blockIdx.x >= b1.nslot;
  const BandTiles& bt = second ? b2 : b1;
  const BandTile t = bt.slot[(int)blockIdx.x - (second ? b1.nslot : 0)];
  double* own = reinterpret_cast<double*>(dyn);
  if (second) band_scale_tile(bt, t, true, own, D2, D1, s2, v2, f2, nullptr);
  else band_scale_tile(bt, t, false, own, D1, D2, s1, v1, f1, rec);
}

__global__ void k_fill(double* __restrict__ a, int64_t na, double* __restrict__ b, int64_t nb, double v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < na) a[i] = v;
  else if (i < na + nb) b[i - na] = v;
}

// Rescaled vectors and the records of their norms: columns (workgroups [0, rc.nblk))
// c_hat = D2 c, l_hat = l / D2, u_hat = u / D2, with |c_hat|_1, |c_hat|_2^2 (sums) and
// |c|_inf (max); rows h_hat = D1 h, with |h_hat|_1, |h_hat|_2^2 and |h|_inf.
__device__ __forceinline__ void scale_vectors(int b, bool rows, const Ranges& R, const double* c, const double* l,
                                              const double* u, const double* h, const double* D1, const double* D2,
                                              const DataMut& d64, const DataMut32& d32, double* rec) {
  __shared__ double lds[kWavesPerBlock * 3];
  double acc[3] = {0.0, 0.0, 0.0};
  const int e1 = R.blk_end[b];
  for (int e = R.blk_start[b] + (int)threadIdx.x; e < e1; e += kBlock) {
    double raw, v;
    if (rows) {
      raw = h[e];
      v = D1[e] * raw;
      d64.h[e] = v;
      d32.h[e] = (float)v;
    } else {
      const double dj = D2[e];
      raw = c[e];
      v = dj * raw;
      const double lv = l[e] / dj, uv = u[e] / dj;
      d64.c[e] = v;
      d64.l[e] = lv;
      d64.u[e] = uv;
      d32.c[e] = (float)v;
      d32.l[e] = (float)lv;
      d32.u[e] = (float)uv;
    }
    acc[0] += fabs(v);
    acc[1] += v * v;
    acc[2] = fmax(acc[2], fabs(raw));
  }
  block_summax_store<3, 2>(acc, lds, rec + (size_t)b * 3);
}

__global__ __launch_bounds__(kBlock) void k_scale_vectors(Ranges rc, Ranges rr, const double* __restrict__ c,
                                                          const double* __restrict__ l, const double* __restrict__ u,
                                                          const double* __restrict__ h, const double* __restrict__ D1,
                                                          const double* __restrict__ D2, DataMut d64, DataMut32 d32,
                                                          double* __restrict__ rec_c, double* __restrict__ rec_r) {
  const bool rows = (int)blockIdx.x >= rc.nblk;
  scale_vectors((int)blockIdx.x - (rows ? rc.nblk : 0), rows, rows ? rr : rc, c, l, u, h, D1, D2, d64, d32,
                rows ? rec_r : rec_c);
}

// Per-instance set-up of the scalars from the norm records (Algorithm 1
// inputs: eta_hat = 1/||G_hat||_inf read as max |G_hat_ij|, primal weight
// initialization of Section 2.5).
__device__ __forceinline__ void init_inst(int iid, const Ranges& rc, const double* rec_c, const Ranges& rr,
                                          const double* rec_r, const int32_t* iblk_m, const double* rec_m, Inst* inst) {
  __shared__ double lds[kWavesPerBlock * 3];
  Inst& I = inst[iid];
  double cs[3], rs[3], ms[1];
  reduce_records<3, 2>(rec_c, rc.inst_blk0[iid], rc.inst_blk0[iid + 1], lds, cs);
  reduce_records<3, 2>(rec_r, rr.inst_blk0[iid], rr.inst_blk0[iid + 1], lds, rs);
  reduce_records<1, 0>(rec_m, iblk_m[iid], iblk_m[iid + 1], lds, ms);
  if (threadIdx.x != 0) return;
  I.c1 = cs[0];
  I.c2 = sqrt(cs[1]);
  I.c_inf = cs[2];
  I.h1 = rs[0];
  I.h2 = sqrt(rs[1]);
  I.h_inf = rs[2];
  I.gmax = ms[0];
  I.eta_hat = ms[0] > 0.0 ? 1.0 / ms[0] : 1.0;
  I.eta = I.eta_hat;
  I.omega0 = (I.c2 > 1e-10 && I.h2 > 1e-10) ? I.c2 / I.h2 : 1.0;
  I.omega = I.omega0;
}

__global__ __launch_bounds__(kBlock) void k_init_inst(Ranges rc, const double* __restrict__ rec_c,
                                                      Ranges rr, const double* __restrict__ rec_r,
                                                      const int32_t* __restrict__ iblk_m,
                                                      const double* __restrict__ rec_m,
                                                      Inst* __restrict__ inst) {
  init_inst(blockIdx.x, rc, rec_c, rr, rec_r, iblk_m, rec_m, inst);
}

// Start point: x = Proj_[l,u](x0 / D2), y = Proj_Kd(y0 / D1); anchor = x_hat = x.
template <typename T>
__device__ __forceinline__ void start_cols(int b, const Ranges& R, const double* x0, const double* D2,
                                           const DataPtrs<double>& d, const IterPtrs<T>& it, double* xs0,
                                           const Inst* inst, int prec) {
  const Inst& I = inst[R.blk_inst[b]];
  if (I.precision != prec) return;
  const int j1 = R.blk_end[b];
  for (int j = R.blk_start[b] + (int)threadIdx.x; j < j1; j += kBlock) {
    const double v = x0 ? x0[j] / D2[j] : 0.0;
    const T x = (T)clampd(v, d.l[j], d.u[j]);
    if (xs0) xs0[j] = (double)x;
    it.x[j] = x;
    it.xa[j] = x;
    it.xh[j] = x;
    it.sx[j] = (T)0;
  }
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_start_cols(Ranges R, const double* __restrict__ x0,
                                                       const double* __restrict__ D2, DataPtrs<double> d,
                                                       IterPtrs<T> it, double* __restrict__ xs0,
                                                       const Inst* __restrict__ inst, int prec) {
  start_cols<T>(blockIdx.x, R, x0, D2, d, it, xs0, inst, prec);
}

template <typename T, bool CONES>
__device__ __forceinline__ void start_rows(int b, const Ranges& R, const double* y0, const double* D1,
                                           const IterPtrs<T>& it, double* ys0, const Inst* inst, int prec) {
  const Inst& I = inst[R.blk_inst[b]];
  if (I.precision != prec) return;
  const int mz_end = I.row0 + I.m_zero;
  const int i1 = R.blk_end[b];
  for (int i = R.blk_start[b] + (int)threadIdx.x; i < i1; i += kBlock) {
    if (i >= I.soc_start) continue;  // cone block rows: below
    const double v = y0 ? y0[i] / D1[i] : 0.0;
    const T y = (T)(i < mz_end ? v : fmax(v, 0.0));
    if (ys0) ys0[i] = (double)y;
    it.y[i] = y;
    it.ya[i] = y;
    it.yh[i] = y;
    it.sy[i] = (T)0;
  }
  // cone blocks: y0 / D1 projected onto diag(1/D1) (dual cone)
  if constexpr (CONES) for_cone_blocks(R, b, [&](auto who, int r0, int dim, int kind) {
    proj_cone(
        who, kind, true, dim, [&](int i) { return y0 ? y0[r0 + i] / D1[r0 + i] : 0.0; }, [&](int i) { return 1.0 / D1[r0 + i]; },
        [&](int i, double p) {
          const int r = r0 + i;
          const T y = (T)p;
          if (ys0) ys0[r] = (double)y;
          it.y[r] = y;
          it.ya[r] = y;
          it.yh[r] = y;
          it.sy[r] = (T)0;
        });
  });
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_start_rows(Ranges R, const double* __restrict__ y0,
                                                       const double* __restrict__ D1, IterPtrs<T> it,
                                                       double* __restrict__ ys0, const Inst* __restrict__ inst,
                                                       int prec) {
  start_rows<T, true>(blockIdx.x, R, y0, D1, it, ys0, inst, prec);
}

// Copy FP64 products into the maintained products of the start point: G^T y (n
// values), then G x (m).
template <typename T>
__global__ void k_set_products(IterPtrs<T> it, const double* __restrict__ gty, int64_t n, const double* __restrict__ gx,
                               int64_t m) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    const T v = (T)gty[i];
    it.gty[i] = v;
    it.gtya[i] = v;
    it.gtyh[i] = v;
  } else if ((i -= n) < m) {
    const T v = (T)gx[i];
    it.gx[i] = v;
    it.gxa[i] = v;
    it.gxh[i] = v;
  }
}

// Plain product out = A in (unscaled or scaled values) for the public SpMV call.
template <typename T, typename TM>
__global__ __launch_bounds__(kBlock) void k_spmv_plain(RowBlocks rb, MatPtrs<TM> A, const T* __restrict__ in,
                                                       T* __restrict__ out) {
  __shared__ double lds[kRowBlockCap + kWavesPerBlock];
  const int b = blockIdx.x;
  const T* const xs[1] = {in};
  block_rows<1>(rb.blk_row0[b], rb.blk_row1[b], A.ptr, A.idx, A.val, xs, lds,
                [&](int r, const double* s) { out[r] = (T)s[0]; });
}

// Instances that fit in LDS (one workgroup each, no cone blocks): what a check, an
// evaluation and the set-up do between two products, in one launch each, with the
// arithmetic of the kernels above and barriers in place of the launches.  Such a
// pass is 1 to 2 us of loads and barriers, a launch of its own 4 to 5 us; the
// products keep theirs, as their row blocks would follow one another here.
// (m = 200, n = 500, 40 trials and one check: 23 launches fewer, 575 -> 531 us a solve;
// 128 LPs of 60 to 220 rows 1605 -> 1560.)
template <typename T>
__device__ __forceinline__ const IterPtrs<T>& iter_of(const KernelCtx& k) {
  if constexpr (sizeof(T) == 4) return k.it32;
  else return k.it64;
}

// After the products of the candidates (of the evaluated point): the candidates'
// sums and their finalizer; then, for an evaluated point, its test and the output,
// and for the start point the products of the iterates.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_cand_wg(KernelCtx k, int prec, int mode) {
  const int iid = blockIdx.x;
  Inst& I = k.inst[iid];
  if (!mode_selects(I, mode) || I.precision != prec) return;  // uniform
  const IterPtrs<T>& it = iter_of<T>(k);
  const int c0 = k.vcol.inst_blk0[iid], c1 = k.vcol.inst_blk0[iid + 1];
  const int r0 = k.vrow.inst_blk0[iid], r1 = k.vrow.inst_blk0[iid + 1];
  for (int b = c0; b < c1; ++b) {
    cand_cols<T>(b, k.vcol, it.xh, it.xbar, it.xa, k.cgty0, k.cgty1, k.d64, k.D2, k.inst, prec, mode, k.rec_cand_c);
    __syncthreads();
  }
  for (int b = r0; b < r1; ++b) {
    cand_rows<T, false>(b, k.vrow, it.yh, it.ybar, it.ya, k.cgx0, k.cgx1, k.d64, k.D1, k.inst, prec, mode, k.rec_cand_r);
    __syncthreads();
  }
  cand_fin(iid, k.vcol, k.rec_cand_c, k.vrow, k.rec_cand_r, k.inst, mode);
  if (mode == kModeCheck) return;
  if (threadIdx.x == 0) eval_fin(I, mode);
  __syncthreads();
  for (int b = c0; b < c1; ++b)
    eval_out<T>(b, true, k.vcol, it.xh, it.yh, k.cgty0, k.d64, k.D1, k.D2, k.xout, k.lamout, k.yout, k.inst, prec, mode);
  for (int b = r0; b < r1; ++b)
    eval_out<T>(b, false, k.vrow, it.xh, it.yh, k.cgty0, k.d64, k.D1, k.D2, k.xout, k.lamout, k.yout, k.inst, prec, mode);
  if (mode != kModeEvalStart) return;
  __syncthreads();
  if (threadIdx.x == 0) eval_start_end(I);
  for (int j = I.col0 + (int)threadIdx.x; j < I.col0 + I.cols; j += kBlock) {
    const T v = (T)k.cgty0[j];
    it.gty[j] = it.gtya[j] = it.gtyh[j] = v;
  }
  for (int i = I.row0 + (int)threadIdx.x; i < I.row0 + I.rows; i += kBlock) {
    const T v = (T)k.cgx0[i];
    it.gx[i] = it.gxa[i] = it.gxh[i] = v;
  }
}

// After the products of the rays: the infeasibility tests, the restart, the end of the check.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_check_wg(KernelCtx k, int prec) {
  const int iid = blockIdx.x;
  Inst& I = k.inst[iid];
  if (I.check_due == 0 || I.precision != prec) return;  // uniform
  const int c0 = k.vcol.inst_blk0[iid], c1 = k.vcol.inst_blk0[iid + 1];
  const int r0 = k.vrow.inst_blk0[iid], r1 = k.vrow.inst_blk0[iid + 1];
  if (mode_selects(I, kModeRay)) {
    for (int b = c0; b < c1; ++b) {
      ray_cols(b, k.vcol, k.ray_x ? k.rx : nullptr, k.rgty, k.d64, k.D2, k.inst, k.rec_cand_c);
      __syncthreads();
    }
    for (int b = r0; b < r1; ++b) {
      ray_rows<false>(b, k.vrow, k.ry, k.ray_x ? k.rgx : nullptr, k.d64, k.D1, k.inst, k.rec_cand_r);
      __syncthreads();
    }
    ray_fin(iid, k.vcol, k.rec_cand_c, k.vrow, k.rec_cand_r, k.inst);
  }
  __syncthreads();
  const IterPtrs<T>& it = iter_of<T>(k);
  for (int b = c0; b < c1; ++b)
    restart_cols<T>(b, k.vcol, it, k.it64, k.cgty0, k.cgty1, k.d64, k.D2, k.xout, k.lamout, k.inst, prec);
  for (int b = r0; b < r1; ++b)
    restart_rows<T>(b, k.vrow, it, k.it64, k.cgx0, k.cgx1, k.D1, k.yout, k.inst, prec);
  __syncthreads();
  if (threadIdx.x == 0) check_end(I);
}

// After the scaling: the rescaled vectors, the instance's scalars, the start point.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_start_wg(KernelCtx k, SetupCtx su, int prec) {
  const int iid = blockIdx.x;
  const IterPtrs<T>& it = iter_of<T>(k);
  const int c0 = k.vcol.inst_blk0[iid], c1 = k.vcol.inst_blk0[iid + 1];
  const int r0 = k.vrow.inst_blk0[iid], r1 = k.vrow.inst_blk0[iid + 1];
  for (int b = c0; b < c1; ++b) {
    scale_vectors(b, false, k.vcol, su.c, su.l, su.u, su.h, k.D1, k.D2, su.d64m, su.d32m, su.rec_nc);
    __syncthreads();
  }
  for (int b = r0; b < r1; ++b) {
    scale_vectors(b, true, k.vrow, su.c, su.l, su.u, su.h, k.D1, k.D2, su.d64m, su.d32m, su.rec_nr);
    __syncthreads();
  }
  init_inst(iid, k.vcol, su.rec_nc, k.vrow, su.rec_nr, k.brow.inst_blk0, su.rec_nm, k.inst);
  for (int b = c0; b < c1; ++b) start_cols<T>(b, k.vcol, su.x0, k.D2, k.d64, it, k.xs0, k.inst, prec);
  for (int b = r0; b < r1; ++b) start_rows<T, false>(b, k.vrow, su.y0, k.D1, it, k.ys0, k.inst, prec);
}

// ===========================================================================
// Launchers
// ===========================================================================
// Whether the instances take the kernels above: the layout runs trials in one
// workgroup per instance and every instance fits in LDS in FP64 (larger ones have
// enough elements for the launches of many workgroups to win).
static inline bool small_instances(const KernelCtx& k) { return k.wg_trials && !k.use_band && k.lds_trials64 > 0; }

static inline dim3 grid1(int n) { return dim3((unsigned)(n > 0 ? n : 0)); }

template <typename T>
static void launch_primal_t(const KernelCtx& k, hipStream_t s, int prec, const IterPtrs<T>& it,
                            const DataPtrs<T>& d) {
  if (k.vcol.nblk > 0)
    k_primal<T><<<grid1(k.vcol.nblk), kBlock, 0, s>>>(k.vcol, it, d, k.inst, prec, k.rec_primal);
}

template <typename T>
static const T* band_val(const KernelCtx& k, int which);
template <>
const float* band_val<float>(const KernelCtx& k, int which) {
  return which ? k.bvalT32 : k.bval32;
}
template <>
const double* band_val<double>(const KernelCtx& k, int which) {
  return which ? k.bvalT64 : k.bval64;
}

// Launches of the band-tile kernels, with the LDS of the layout's accumulators.
template <typename T>
static void launch_band_spmv(const BandTiles& bt, const T* val, const T* x, T* part, int64_t R, const Inst* inst, int prec,
                             int need_acc, int idle, hipStream_t s) {
  if (bt.nslot > 0)
    k_band_spmv<T><<<grid1(bt.nslot), kWave, (size_t)bt.slots * sizeof(T), s>>>(
        bt, val, x, part, R, inst, prec, need_acc, idle);
}

template <typename TX>
static void launch_band_cand(const BandTiles& bt, const double* val, const TX* x, double* part, int64_t R,
                             const Inst* inst, int prec, int mode, int which, hipStream_t s) {
  if (bt.nslot > 0)
    k_band_cand<TX><<<grid1(bt.nslot), kWave, (size_t)bt.slots * 8, s>>>(
        bt, val, x, part, R, inst, prec, mode, which);
}

// Lets the band-tile kernels ask for up to kBandSlots FP64 accumulators per
// wave on the current device.
hipError_t band_raise_lds_limit() {
  const void* const fns[] = {reinterpret_cast<const void*>(&k_band_spmv<float>), reinterpret_cast<const void*>(&k_band_spmv<double>),
                             reinterpret_cast<const void*>(&k_band_cand<float>), reinterpret_cast<const void*>(&k_band_cand<double>),
                             reinterpret_cast<const void*>(&k_band_lam_fold<float, false>), reinterpret_cast<const void*>(&k_band_lam_fold<float, true>), reinterpret_cast<const void*>(&k_band_lam_fold<double, false>), reinterpret_cast<const void*>(&k_band_lam_fold<double, true>),
                             reinterpret_cast<const void*>(&k_scale_bands<MaxProduct>),
                             reinterpret_cast<const void*>(&k_scale_bands<SumSquares>),
                             reinterpret_cast<const void*>(&k_scale_bands_values)};
  for (const void* f : fns) {
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kBandSlots * 8);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <typename T>
static void launch_dual_t(const KernelCtx& k, hipStream_t s, int prec, const IterPtrs<T>& it,
                          const DataPtrs<T>& d, const MatPtrs<T>& A, T* part) {
  if (k.use_band) {
    launch_band_spmv<T>(k.band1, band_val<T>(k, 0), it.xh, part, k.M, k.inst, prec, 0, k.idle, s);
  } else if (k.brow.nblk > 0) {
    k_dual<T, T><<<grid1(k.brow.nblk), kBlock, 0, s>>>(k.brow, A, it, d, k.inst, prec, k.rec_dual);
  }
}

template <typename T>
static void launch_dual_epi_t(const KernelCtx& k, hipStream_t s, int prec, const IterPtrs<T>& it,
                              const DataPtrs<T>& d, const T* part) {
  if (k.use_band && k.vrow.nblk > 0)
    k_dual_epi<T><<<grid1(k.vrow.nblk), kBlock, 0, s>>>(k.vrow, part, k.band1.P, k.M, it, d,
                                                         k.D1, k.inst, prec, k.rec_dual_epi);
}

template <typename T>
static void launch_lam_t(const KernelCtx& k, hipStream_t s, int prec, const IterPtrs<T>& it,
                         const DataPtrs<T>& d, const MatPtrs<T>& AT, T* part) {
  if (k.use_band) {
    launch_band_spmv<T>(k.band2, band_val<T>(k, 1), it.yh, part, k.N, k.inst, prec, 1, k.idle, s);
    if (k.vcol.nblk > 0)
      k_lam_epi<T><<<grid1(k.vcol.nblk), kBlock, 0, s>>>(k.vcol, part, k.band2.P, k.N, it, d, k.inst, prec,
                                                          k.rec_lam_epi);
  } else if (k.bcol.nblk > 0) {
    k_lam<T, T><<<grid1(k.bcol.nblk), kBlock, 0, s>>>(k.bcol, AT, it, d, k.inst, prec, k.rec_lam);
  }
}

// part 0: primal pass; part 1: the SpMV G x_hat (fused with the dual step on
// row blocks; band tiles write partial sums); part 2: the rest of the trial.
void launch_trial_part(const KernelCtx& k, hipStream_t s, int mask, int part) {
  if (part == 0) {
    if (mask & 1) launch_primal_t<float>(k, s, kFP32, k.it32, k.d32);
    if (mask & 2) launch_primal_t<double>(k, s, kFP64, k.it64, k.d64);
    return;
  }
  if (part == 1) {
    if (mask & 1) launch_dual_t<float>(k, s, kFP32, k.it32, k.d32, k.A32, k.bpart32);
    if (mask & 2) launch_dual_t<double>(k, s, kFP64, k.it64, k.d64, k.A64, k.bpart64);
    return;
  }
  if (mask & 1) launch_dual_epi_t<float>(k, s, kFP32, k.it32, k.d32, k.bpart32);
  if (mask & 2) launch_dual_epi_t<double>(k, s, kFP64, k.it64, k.d64, k.bpart64);
  const bool split = k.use_band != 0;
  k_fin_ls<<<grid1(k.nb), kBlock, 0, s>>>(k.vcol.inst_blk0, k.rec_primal,
                                           split ? k.vrow.inst_blk0 : k.brow.inst_blk0,
                                           split ? k.rec_dual_epi : k.rec_dual, k.inst);
  if (mask & 1) launch_lam_t<float>(k, s, kFP32, k.it32, k.d32, k.AT32, k.bpartT32);
  if (mask & 2) launch_lam_t<double>(k, s, kFP64, k.it64, k.d64, k.AT64, k.bpartT64);
  k_fin_beta<<<grid1(k.nb), kBlock, 0, s>>>(split ? k.vcol.inst_blk0 : k.bcol.inst_blk0,
                                             split ? k.rec_lam_epi : k.rec_lam, k.inst);
}

// K trials with the finalizers folded into the passes (k.fold): the instance
// records alternate between inst and inst2 and are back in inst at the end.
template <typename T, bool IDLE>
static void launch_primal_fold_t(const KernelCtx& k, hipStream_t s, int prec, const IterPtrs<T>& it,
                                 const DataPtrs<T>& d, const FoldIn& f) {
  if (k.vcol.nblk > 0) k_primal_fold<T, IDLE><<<grid1(k.vcol.nblk), kBlock, 0, s>>>(k.vcol, it, d, f, prec, k.rec_primal);
}

template <typename T, bool IDLE>
static void launch_lam_fold_t(const KernelCtx& k, hipStream_t s, int prec, const IterPtrs<T>& it, const DataPtrs<T>& d,
                              const MatPtrs<T>& AT, T* part, const FoldIn& f) {
  if (k.use_band && k.band_lam) {
    if (k.band2.nslot > 0)
      k_band_lam_fold<T, IDLE><<<grid1(k.band2.nslot + k.nb), kWave, (size_t)k.band2.slots * sizeof(T), s>>>(
          k.band2, band_val<T>(k, 1), it, d, f, prec, k.rec_lam_epi);
  } else if (k.use_band) {
    // (whether the trial is accepted is not known yet: the product runs either way, 30 to
    // 35 us for a rejected trial of 4.7e6 nonzeros, where every trial saves 4.7 of 106; see k_lam_fold)
    launch_band_spmv<T>(k.band2, band_val<T>(k, 1), it.yh, part, k.N, k.inst, prec, 0, k.idle, s);
    if (k.vcol.nblk > 0)
      k_lam_epi_fold<T, IDLE><<<grid1(k.vcol.nblk), kBlock, 0, s>>>(k.vcol, part, k.band2.P, k.N, it, d, f, prec,
                                                               k.rec_lam_epi);
  } else if (k.bcol.nblk > 0) {
    k_lam_fold<T, T, IDLE><<<grid1(k.bcol.nblk), kBlock, 0, s>>>(k.bcol, AT, it, d, f, prec, k.rec_lam);
  }
}

template <bool IDLE>
static void launch_trials_fold_t(const KernelCtx& k, hipStream_t s, int mask, int K) {
  const bool split = k.use_band != 0;
  const FoldIn ls{k.vcol.inst_blk0, split ? k.vrow.inst_blk0 : k.brow.inst_blk0, k.rec_primal,
                  split ? k.rec_dual_epi : k.rec_dual, k.inst, k.inst2};
  const FoldIn beta{split ? (k.band_lam ? k.band2_tile0 : k.vcol.inst_blk0) : k.bcol.inst_blk0, nullptr, split ? k.rec_lam_epi : k.rec_lam, nullptr,
                    k.inst2, k.inst};
  for (int t = 0; t < K; ++t) {
    if (t == 0) {
      launch_trial_part(k, s, mask, 0);
    } else {
      if (mask & 1) launch_primal_fold_t<float, IDLE>(k, s, kFP32, k.it32, k.d32, beta);
      if (mask & 2) launch_primal_fold_t<double, IDLE>(k, s, kFP64, k.it64, k.d64, beta);
    }
    launch_trial_part(k, s, mask, 1);
    if (mask & 1) launch_dual_epi_t<float>(k, s, kFP32, k.it32, k.d32, k.bpart32);
    if (mask & 2) launch_dual_epi_t<double>(k, s, kFP64, k.it64, k.d64, k.bpart64);
    if (mask & 1) launch_lam_fold_t<float, IDLE>(k, s, kFP32, k.it32, k.d32, k.AT32, k.bpartT32, ls);
    if (mask & 2) launch_lam_fold_t<double, IDLE>(k, s, kFP64, k.it64, k.d64, k.AT64, k.bpartT64, ls);
  }
  if (K > 0) k_fold_end<<<grid1(k.nb), kBlock, 0, s>>>(beta);
}

void launch_trials_fold(const KernelCtx& k, hipStream_t s, int mask, int K) {
  if (k.idle) launch_trials_fold_t<true>(k, s, mask, K);
  else launch_trials_fold_t<false>(k, s, mask, K);
}

// Dynamic LDS the LDS-resident chunk kernel can take: the device's LDS per
// workgroup less the most static LDS of the kernels that get it (both forms of
// that kernel and, in FP64, the set-up's); the first call per precision also
// raises these kernels' dynamic-LDS limits to that size.
template <typename T>
static size_t lds_capacity_t() {
  static size_t cap = 0;
  static bool done = false;
  if (!done) {
    done = true;
    int dev = 0, max_lds = 0, optin = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) == hipSuccess) {
      if (hipDeviceGetAttribute(&optin, hipDeviceAttributeSharedMemPerBlockOptin, dev) == hipSuccess)
        max_lds = std::max(max_lds, optin);
    }
    const void* kernels[3] = {reinterpret_cast<const void*>(&k_trials_lds<T, kBlock>),
                              reinterpret_cast<const void*>(&k_trials_lds<T, kRowThreads>),
                              reinterpret_cast<const void*>(&k_scale_lds)};
    const int count = std::is_same_v<T, double> ? 3 : 2;
    size_t fixed = 1024;
    bool ok = max_lds > 0;
    for (int i = 0; i < count && ok; ++i) {
      hipFuncAttributes fa{};
      ok = hipFuncGetAttributes(&fa, kernels[i]) == hipSuccess;
      fixed = std::max(fixed, fa.sharedSizeBytes + 1024);
    }
    ok = ok && (size_t)max_lds > fixed;
    for (int i = 0; i < count && ok; ++i)
      ok = hipFuncSetAttribute(kernels[i], hipFuncAttributeMaxDynamicSharedMemorySize, (int)(max_lds - fixed)) == hipSuccess;
    if (ok) cap = (size_t)max_lds - fixed;
    (void)hipGetLastError();
  }
  return cap;
}

size_t trials_lds_capacity(int prec) { return prec == kFP32 ? lds_capacity_t<float>() : lds_capacity_t<double>(); }

template <typename T>
static void launch_trials_wg_t(const KernelCtx& k, hipStream_t s, int prec, int K, int lds, const MatPtrs<T>& A,
                               const MatPtrs<T>& AT, const IterPtrs<T>& it, const DataPtrs<T>& d) {
  if (lds > 0 && k.lds_rowwise)
    k_trials_lds<T, kRowThreads><<<k.nb, kRowThreads, lds, s>>>(k.vcol, k.brow, k.bcol, A, AT, it, d, k.inst, prec, K);
  else if (lds > 0)
    k_trials_lds<T, kBlock><<<k.nb, kBlock, lds, s>>>(k.vcol, k.brow, k.bcol, A, AT, it, d, k.inst, prec, K);
  else
    k_trials_wg<T><<<k.nb, kBlock, 0, s>>>(k.vcol, k.brow, k.bcol, A, AT, it, d, k.inst, prec, k.rec_primal, k.rec_dual,
                                           k.rec_lam, K);
}

void launch_trials_wg(const KernelCtx& k, hipStream_t s, int mask, int K) {
  if (k.nb < 1 || K < 1) return;
  if (mask & 1) launch_trials_wg_t<float>(k, s, kFP32, K, k.lds_trials32, k.A32, k.AT32, k.it32, k.d32);
  if (mask & 2) launch_trials_wg_t<double>(k, s, kFP64, K, k.lds_trials64, k.A64, k.AT64, k.it64, k.d64);
}

template <typename T>
static void launch_cand_t(const KernelCtx& k, hipStream_t s, int prec, const IterPtrs<T>& it,
                          const T* x0, const T* x1, const T* y0, const T* y1, int mode) {
  if (small_instances(k)) {
    if (k.bcol.nblk + k.brow.nblk > 0)
      k_spmv2<T><<<grid1(k.bcol.nblk + k.brow.nblk), kBlock, 0, s>>>(
          Spmv2Side<T>{k.bcol, k.AT64, y0, y1, k.cgty0, k.cgty1}, Spmv2Side<T>{k.brow, k.A64, x0, x1, k.cgx0, k.cgx1},
          k.inst, prec, mode);
    k_cand_wg<T><<<grid1(k.nb), kBlock, 0, s>>>(k, prec, mode);
    return;
  }
  if (k.use_band) {
    // band tiles with FP64 values: one pass per vector, then the window sums
    launch_band_cand<T>(k.band1, k.bval64, x0, k.bpart64, k.M, k.inst, prec, mode, 0, s);
    if (x1) launch_band_cand<T>(k.band1, k.bval64, x1, k.bpart64b, k.M, k.inst, prec, mode, 1, s);
    launch_band_cand<T>(k.band2, k.bvalT64, y0, k.bpartT64, k.N, k.inst, prec, mode, 0, s);
    if (y1) launch_band_cand<T>(k.band2, k.bvalT64, y1, k.bpartT64b, k.N, k.inst, prec, mode, 1, s);
    if (k.vcol.nblk + k.vrow.nblk > 0)
      k_band_combine2<<<grid1(k.vcol.nblk + k.vrow.nblk), kBlock, 0, s>>>(
          CombineSide{k.vcol, k.band2.P, k.N, k.bpartT64, y1 ? k.bpartT64b : nullptr, k.cgty0, k.cgty1},
          CombineSide{k.vrow, k.band1.P, k.M, k.bpart64, x1 ? k.bpart64b : nullptr, k.cgx0, k.cgx1}, k.inst, mode);
  } else if (k.bcol.nblk + k.brow.nblk > 0) {
    k_spmv2<T><<<grid1(k.bcol.nblk + k.brow.nblk), kBlock, 0, s>>>(
        Spmv2Side<T>{k.bcol, k.AT64, y0, y1, k.cgty0, k.cgty1}, Spmv2Side<T>{k.brow, k.A64, x0, x1, k.cgx0, k.cgx1},
        k.inst, prec, mode);
  }
  if (k.vcol.nblk > 0)
    k_cand_cols<T><<<grid1(k.vcol.nblk), kBlock, 0, s>>>(k.vcol, x0, x1, it.xa, k.cgty0, k.cgty1, k.d64, k.D2,
                                                          k.inst, prec, mode, k.rec_cand_c);
  if (k.vrow.nblk > 0)
    k_cand_rows<T><<<grid1(k.vrow.nblk), kBlock, 0, s>>>(k.vrow, y0, y1, it.ya, k.cgx0, k.cgx1, k.d64, k.D1,
                                                          k.inst, prec, mode, k.rec_cand_r);
}

template <typename T>
static void launch_check_pre_t(const KernelCtx& k, hipStream_t s, int prec, const IterPtrs<T>& it) {
  if (k.vcol.nblk + k.vrow.nblk > 0)
    k_commit_avg<T><<<grid1(k.vcol.nblk + k.vrow.nblk), kBlock, 0, s>>>(commit_cols(k.vcol, it), commit_rows(k.vrow, it),
                                                                         k.inst, prec);
  launch_cand_t<T>(k, s, prec, it, it.xh, it.xbar, it.yh, it.ybar, kModeCheck);
}

template <typename T>
static void launch_probe_t(const KernelCtx& k, hipStream_t s, int prec, const IterPtrs<T>& it) {
  if (k.ccol.nblk + k.crow.nblk > 0)
    k_probe<T><<<dim3(k.ccol.nblk + k.crow.nblk, kMaxCand), kBlock, 0, s>>>(
        k.ccol, k.crow, it.xh, it.xbar, it.yh, it.ybar, k.cgty0, k.cgty1, k.cgx0, k.cgx1, k.d64, k.D1, k.inst, prec,
        k.rec_probe_c, k.rec_probe_r);
}

template <typename T>
static void launch_probes_wg_t(const KernelCtx& k, hipStream_t s, int prec, const IterPtrs<T>& it) {
  k_probes_wg<T><<<k.nb, kProbeGroups * kBlock, 0, s>>>(it.xh, it.xbar, it.yh, it.ybar, k.cgty0, k.cgty1, k.cgx0, k.cgx1,
                                                        k.d64, k.inst, prec, k.probe_passes,
                                                        RayOut{k.xs0, k.ys0, k.ray_x ? k.rx : nullptr, k.ry});
}

template <typename T>
static void launch_restart_t(const KernelCtx& k, hipStream_t s, int prec, const IterPtrs<T>& it) {
  if (k.vcol.nblk + k.vrow.nblk > 0)
    k_restart<T><<<grid1(k.vcol.nblk + k.vrow.nblk), kBlock, 0, s>>>(k.vcol, k.vrow, it, k.it64, k.cgty0, k.cgty1, k.cgx0,
                                                                      k.cgx1, k.d64, k.D1, k.D2, k.xout, k.lamout,
                                                                      k.yout, k.inst, prec);
}

// Products of the rays with FP64 values (every selected instance, whatever
// its precision): rgty = G_hat^T r_y, and rgx = G_hat r_x when some instance
// has an unbounded column.
static void launch_ray_products(const KernelCtx& k, hipStream_t s) {
  if (k.use_band) {
    launch_band_cand<double>(k.band2, k.bvalT64, k.ry, k.bpartT64, k.N, k.inst, kFP64, kModeRay, 0, s);
    if (k.ray_x) launch_band_cand<double>(k.band1, k.bval64, k.rx, k.bpart64, k.M, k.inst, kFP64, kModeRay, 0, s);
    Ranges rows = k.vrow;
    if (!k.ray_x) rows.nblk = 0;
    if (k.vcol.nblk + rows.nblk > 0)
      k_band_combine2<<<grid1(k.vcol.nblk + rows.nblk), kBlock, 0, s>>>(
          CombineSide{k.vcol, k.band2.P, k.N, k.bpartT64, nullptr, k.rgty, nullptr},
          CombineSide{rows, k.band1.P, k.M, k.bpart64, nullptr, k.rgx, nullptr}, k.inst, kModeRay);
    return;
  }
  RowBlocks rows = k.brow;
  if (!k.ray_x) rows.nblk = 0;
  if (k.bcol.nblk + rows.nblk > 0)
    k_spmv2<double><<<grid1(k.bcol.nblk + rows.nblk), kBlock, 0, s>>>(
        Spmv2Side<double>{k.bcol, k.AT64, k.ry, nullptr, k.rgty, nullptr},
        Spmv2Side<double>{rows, k.A64, k.rx, nullptr, k.rgx, nullptr}, k.inst, kFP64, kModeRay);
}

template <typename T>
static void launch_ray_vec_t(const KernelCtx& k, hipStream_t s, int prec, const IterPtrs<T>& it) {
  if (k.vcol.nblk > 0 && k.ray_x)
    k_ray_vec_cols<T><<<grid1(k.vcol.nblk), kBlock, 0, s>>>(k.vcol, it.xh, k.xs0, k.d64, k.rx, k.inst, prec);
  if (k.vrow.nblk > 0)
    k_ray_vec_rows<T><<<grid1(k.vrow.nblk), kBlock, 0, s>>>(k.vrow, it.yh, k.ys0, k.D1, k.ry, k.inst, prec);
}

// The infeasibility tests of one check (instances selected by k_decide).
static void launch_ray(const KernelCtx& k, hipStream_t s, int mask) {
  if (!k.wg_trials || k.use_band) {  // (else with the multisection passes)
    if (mask & 1) launch_ray_vec_t<float>(k, s, kFP32, k.it32);
    if (mask & 2) launch_ray_vec_t<double>(k, s, kFP64, k.it64);
  }
  launch_ray_products(k, s);
  // the candidate records are free once k_cand_fin has run
  if (k.vcol.nblk > 0)
    k_ray_cols<<<grid1(k.vcol.nblk), kBlock, 0, s>>>(k.vcol, k.ray_x ? k.rx : nullptr, k.rgty, k.d64, k.D2, k.inst,
                                                      k.rec_cand_c);
  if (k.vrow.nblk > 0)
    k_ray_rows<<<grid1(k.vrow.nblk), kBlock, 0, s>>>(k.vrow, k.ry, k.ray_x ? k.rgx : nullptr, k.d64, k.D1, k.inst,
                                                      k.rec_cand_r);
  k_ray_fin<<<grid1(k.nb), kBlock, 0, s>>>(k.vcol, k.rec_cand_c, k.vrow, k.rec_cand_r, k.inst);
}

void launch_check(const KernelCtx& k, hipStream_t s, int mask) {
  const int nbt = (k.nb + 63) / 64;
  if (mask & 1) launch_check_pre_t<float>(k, s, kFP32, k.it32);
  if (mask & 2) launch_check_pre_t<double>(k, s, kFP64, k.it64);
  const bool small = small_instances(k);
  if (!small)
    k_cand_fin<<<grid1(k.nb), kBlock, 0, s>>>(k.vcol, k.rec_cand_c, k.vrow, k.rec_cand_r, k.inst, kModeCheck);
  if (k.wg_trials && !k.use_band) {
    if (mask & 1) launch_probes_wg_t<float>(k, s, kFP32, k.it32);
    if (mask & 2) launch_probes_wg_t<double>(k, s, kFP64, k.it64);
  } else {
    for (int pass = 0; pass < k.probe_passes; ++pass) {
      if (mask & 1) launch_probe_t<float>(k, s, kFP32, k.it32);
      if (mask & 2) launch_probe_t<double>(k, s, kFP64, k.it64);
      k_probe_fin<<<grid1(k.nb), kProbeGroups * kBlock, 0, s>>>(k.ccol, k.rec_probe_c, k.crow, k.rec_probe_r, k.inst);
    }
    k_decide<<<nbt, 64, 0, s>>>(k.inst, k.nb);
  }
  if (small) {
    if (k.infeas) launch_ray_products(k, s);
    if (mask & 1) k_check_wg<float><<<grid1(k.nb), kBlock, 0, s>>>(k, kFP32);
    if (mask & 2) k_check_wg<double><<<grid1(k.nb), kBlock, 0, s>>>(k, kFP64);
    return;
  }
  if (k.infeas) launch_ray(k, s, mask);
  if (mask & 1) launch_restart_t<float>(k, s, kFP32, k.it32);
  if (mask & 2) launch_restart_t<double>(k, s, kFP64, k.it64);
  k_check_end<<<nbt, 64, 0, s>>>(k.inst, k.nb);
}

void launch_summary(const KernelCtx& k, hipStream_t s, int32_t* out) {
  k_summary<<<1, kBlock, 0, s>>>(k.inst, k.nb, out);
}

void launch_timeout(const KernelCtx& k, hipStream_t s) {
  k_timeout<<<(k.nb + 63) / 64, 64, 0, s>>>(k.inst, k.nb);
}

template <typename T>
static void launch_eval_t(const KernelCtx& k, hipStream_t s, int prec, const IterPtrs<T>& it, int mode) {
  launch_cand_t<T>(k, s, prec, it, it.xh, nullptr, it.yh, nullptr, mode);
}

template <typename T>
static void launch_eval_out_t(const KernelCtx& k, hipStream_t s, int prec, const IterPtrs<T>& it, int mode) {
  if (k.vcol.nblk + k.vrow.nblk > 0)
    k_eval_out<T><<<grid1(k.vcol.nblk + k.vrow.nblk), kBlock, 0, s>>>(k.vcol, k.vrow, it.xh, it.yh, k.cgty0, k.d64, k.D1,
                                                                       k.D2, k.xout, k.lamout, k.yout, k.inst, prec, mode);
}

void launch_eval(const KernelCtx& k, hipStream_t s, int mask, int final_mode) {
  const int mode = final_mode ? kModeEvalFinal : kModeEvalStart;
  const int nbt = (k.nb + 63) / 64;
  if (mask & 1) launch_eval_t<float>(k, s, kFP32, k.it32, mode);
  if (mask & 2) launch_eval_t<double>(k, s, kFP64, k.it64, mode);
  if (small_instances(k)) return;
  k_cand_fin<<<grid1(k.nb), kBlock, 0, s>>>(k.vcol, k.rec_cand_c, k.vrow, k.rec_cand_r, k.inst, mode);
  k_eval_fin<<<nbt, 64, 0, s>>>(k.inst, k.nb, mode);
  if (mask & 1) launch_eval_out_t<float>(k, s, kFP32, k.it32, mode);
  if (mask & 2) launch_eval_out_t<double>(k, s, kFP64, k.it64, mode);
  if (!final_mode) k_eval_start_end<<<nbt, 64, 0, s>>>(k.inst, k.nb);
}

template <typename T>
static void launch_flush_t(const KernelCtx& k, hipStream_t s, int prec, const IterPtrs<T>& it) {
  if (k.vcol.nblk > 0)
    k_flush_commit<T><<<grid1(k.vcol.nblk), kBlock, 0, s>>>(k.vcol, it.x, it.xh, it.xa, it.gty, it.gtyh,
                                                             it.gtya, it.sx, k.inst, prec);
  if (k.vrow.nblk > 0)
    k_flush_commit<T><<<grid1(k.vrow.nblk), kBlock, 0, s>>>(k.vrow, it.y, it.yh, it.ya, it.gx, it.gxh, it.gxa,
                                                             it.sy, k.inst, prec);
}

void launch_flush_commit(const KernelCtx& k, hipStream_t s, int mask) {
  if (mask & 1) launch_flush_t<float>(k, s, kFP32, k.it32);
  if (mask & 2) launch_flush_t<double>(k, s, kFP64, k.it64);
  k_clear_pending<<<(k.nb + 63) / 64, 64, 0, s>>>(k.inst, k.nb);
}

// ---- set-up ----
static ScaleSide scale_side(const KernelCtx& k, const SetupCtx& su, int cols, const double* D1, const double* D2) {
  return cols ? ScaleSide{k.bcol, su.AT.ptr, su.AT.idx, su.AT.val, D2, D1, 1}
              : ScaleSide{k.brow, su.A.ptr, su.A.idx, su.A.val, D1, D2, 0};
}

void launch_scale_values(const KernelCtx& k, const SetupCtx& su, hipStream_t s, double* rec) {
  const unsigned nblk = (unsigned)(k.brow.nblk + k.bcol.nblk);
  if (nblk > 0)
    k_scale_values<<<nblk, kBlock, 0, s>>>(scale_side(k, su, 0, k.D1, k.D2), scale_side(k, su, 1, k.D1, k.D2), su.val64,
                                           su.val32, su.valT64, su.valT32, rec);
}

void launch_setup(const KernelCtx& k, const SetupCtx& su, hipStream_t s, int mask) {
  const int tpb = 256;
  auto blocks = [&](int64_t n) { return dim3((unsigned)((n + tpb - 1) / tpb)); };
  const int passes = su.precondition ? su.ruiz_iters + (su.l2_pass ? 1 : 0) : 0;
  if (k.use_band) {
    const unsigned slots = (unsigned)(k.band1.nslot + k.band2.nslot);
    double *d1[2] = {k.D1, su.stat_r}, *d2[2] = {k.D2, su.stat_c};  // the last pass writes D1, D2
    const int odd = slots > 0 ? passes & 1 : 0;
    k_fill<<<blocks(k.M + k.N), tpb, 0, s>>>(d1[odd], k.M, d2[odd], k.N, 1.0);
    const size_t lds = (size_t)std::max(k.band1.slots, k.band2.slots) * 8;
    const double *v1 = su.borig64, *v2 = su.borigT64;
    if (!v1) {  // a batch keeps no unscaled values in entry order: they pass through the scaled ones' place
      if (su.bn > 0) launch_band_vals(su.bsrc, su.bn, su.A.val, su.bval64, su.bval32, s);
      if (su.bnT > 0) launch_band_vals(su.bsrcT, su.bnT, su.AT.val, su.bvalT64, su.bvalT32, s);
      v1 = su.bval64, v2 = su.bvalT64;
    }
    if (slots > 0) {
      for (int i = 0; i < passes; ++i) {
        const int mode = i < su.ruiz_iters ? kScaleMax : kScaleSquares;
        const int to = (passes - 1 - i) & 1;
        if (mode == kScaleMax)
          k_scale_bands<MaxProduct><<<slots, kWave, lds, s>>>(k.band1, v1, d2[!to], k.bpart64, k.M, k.band2, v2, d1[!to],
                                                              k.bpartT64, k.N);
        else
          k_scale_bands<SumSquares><<<slots, kWave, lds, s>>>(k.band1, v1, d2[!to], k.bpart64, k.M, k.band2, v2, d1[!to],
                                                              k.bpartT64, k.N);
        k_scale_bands_update<<<blocks(k.M + k.N), tpb, 0, s>>>(
            scale_side(k, su, 0, d1[!to], d2[!to]), scale_side(k, su, 1, d1[!to], d2[!to]), k.bpart64, k.band1.P, k.M,
            k.bpartT64, k.band2.P, k.N, mode, d1[to], d2[to]);
      }
      k_scale_bands_values<<<slots, kWave, lds, s>>>(k.band1, v1, su.bval64, su.bval32, k.band2, v2,
                                                                  su.bvalT64, su.bvalT32, k.D1, k.D2, su.rec_nm);
    }
  } else if (k.lds_trials64 > 0 && k.lds_rowwise) {
    k_scale_lds<<<k.nb, kScaleLdsThreads, k.lds_trials64, s>>>(su.A, su.AT, k.brow.inst_blk0, passes, su.ruiz_iters, k.D1,
                                                               k.D2, su.val64, su.val32, su.valT64, su.valT32, k.inst,
                                                               su.rec_nm);
  } else {
    const unsigned nblk = (unsigned)(k.brow.nblk + k.bcol.nblk);
    if (passes == 0) k_fill<<<blocks(k.M + k.N), tpb, 0, s>>>(k.D1, k.M, k.D2, k.N, 1.0);
    double *d1[2] = {k.D1, su.stat_r}, *d2[2] = {k.D2, su.stat_c};  // the last pass writes D1, D2
    for (int i = 0; i < passes; ++i) {
      const int to = (passes - 1 - i) & 1;
      k_scale_pass<<<nblk, kBlock, 0, s>>>(
          scale_side(k, su, 0, i ? d1[!to] : nullptr, i ? d2[!to] : nullptr),
          scale_side(k, su, 1, i ? d1[!to] : nullptr, i ? d2[!to] : nullptr),
          i < su.ruiz_iters ? kScaleMax : kScaleSquares, d1[to], d2[to]);
    }
    launch_scale_values(k, su, s, su.rec_nm);
  }
  if (small_instances(k) && (mask == 1 || mask == 2)) {
    if (mask == 1) k_start_wg<float><<<grid1(k.nb), kBlock, 0, s>>>(k, su, kFP32);
    else k_start_wg<double><<<grid1(k.nb), kBlock, 0, s>>>(k, su, kFP64);
    launch_eval(k, s, mask, 0);
    return;
  }
  k_scale_vectors<<<grid1(k.vcol.nblk + k.vrow.nblk), kBlock, 0, s>>>(k.vcol, k.vrow, su.c, su.l, su.u, su.h, k.D1, k.D2,
                                                                      su.d64m, su.d32m, su.rec_nc, su.rec_nr);
  k_init_inst<<<grid1(k.nb), kBlock, 0, s>>>(k.vcol, su.rec_nc, k.vrow, su.rec_nr,
                                             k.use_band ? su.btile0 : k.brow.inst_blk0, su.rec_nm, k.inst);
  // start point and its products
  if (mask & 1) {
    if (k.vcol.nblk > 0)
      k_start_cols<float><<<grid1(k.vcol.nblk), kBlock, 0, s>>>(k.vcol, su.x0, k.D2, k.d64, k.it32, k.xs0, k.inst,
                                                                 kFP32);
    if (k.vrow.nblk > 0)
      k_start_rows<float><<<grid1(k.vrow.nblk), kBlock, 0, s>>>(k.vrow, su.y0, k.D1, k.it32, k.ys0, k.inst, kFP32);
  }
  if (mask & 2) {
    if (k.vcol.nblk > 0)
      k_start_cols<double><<<grid1(k.vcol.nblk), kBlock, 0, s>>>(k.vcol, su.x0, k.D2, k.d64, k.it64, k.xs0, k.inst,
                                                                  kFP64);
    if (k.vrow.nblk > 0)
      k_start_rows<double><<<grid1(k.vrow.nblk), kBlock, 0, s>>>(k.vrow, su.y0, k.D1, k.it64, k.ys0, k.inst, kFP64);
  }
  // FP64-value products of the start point: eval mode computes cgx0 = G x_hat, cgty0 = G^T y_hat
  launch_eval(k, s, mask, 0);
  if (small_instances(k)) return;
  if (mask & 1) k_set_products<float><<<blocks(k.M + k.N), tpb, 0, s>>>(k.it32, k.cgty0, k.N, k.cgx0, k.M);
  if (mask & 2) k_set_products<double><<<blocks(k.M + k.N), tpb, 0, s>>>(k.it64, k.cgty0, k.N, k.cgx0, k.M);
}

void launch_spmv_plain(const RowBlocks& rb, int prec, const int32_t* ptr, const int32_t* idx, const void* val,
                       const void* in, void* out, hipStream_t s) {
  if (rb.nblk <= 0) return;
  if (prec == kFP64) {
    MatPtrs<double> A{ptr, idx, (const double*)val};
    k_spmv_plain<double, double><<<grid1(rb.nblk), kBlock, 0, s>>>(rb, A, (const double*)in, (double*)out);
  } else {
    MatPtrs<float> A{ptr, idx, (const float*)val};
    k_spmv_plain<float, float><<<grid1(rb.nblk), kBlock, 0, s>>>(rb, A, (const float*)in, (float*)out);
  }
}

// One K1 pass on its own (for schedule timing).
void launch_band_plain(const BandTiles& bt, int prec, const void* val, const void* in, void* part, int64_t R,
                       void* out, hipStream_t s) {
  if (bt.nslot <= 0 || R <= 0) return;
  const dim3 g((unsigned)((R + 255) / 256));
  if (prec == kFP64) {
    launch_band_spmv<double>(bt, (const double*)val, (const double*)in, (double*)part, R, nullptr, kFP64, 0, 0, s);
    k_band_sum<double><<<g, 256, 0, s>>>((const double*)part, bt.P, R, (double*)out);
  } else {
    launch_band_spmv<float>(bt, (const float*)val, (const float*)in, (float*)part, R, nullptr, kFP32, 0, 0, s);
    k_band_sum<float><<<g, 256, 0, s>>>((const float*)part, bt.P, R, (float*)out);
  }
}

void launch_band_vals(const int32_t* src, int64_t n, const double* v64, double* o64, float* o32, hipStream_t s) {
  if (n > 0) k_band_vals<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(src, n, v64, o64, o32);
}

__global__ void k_to_f32(const double* __restrict__ in, float* __restrict__ out, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    out[i] = (float)in[i];
}

void launch_to_f32(const double* in, float* out, int64_t n, hipStream_t s) {
  if (n > 0) k_to_f32<<<(unsigned)std::min<int64_t>((n + 255) / 256, 65536), 256, 0, s>>>(in, out, n);
}

void launch_copies(const CopyItem* items, size_t count, hipStream_t s) {
  for (size_t i = 0; i < count;) {
    CopyList list;
    int64_t longest = 0;
    int k = 0;
    for (; i < count && k < kCopyList; ++i)
      if (items[i].len > 0) {
        list.item[k++] = items[i];
        longest = std::max(longest, items[i].len);
      }
    if (k > 0)
      k_copies<<<dim3((unsigned)std::min<int64_t>((longest + 4 * kBlock - 1) / (4 * kBlock), 256), (unsigned)k), kBlock, 0,
                 s>>>(list);
  }
}

void launch_proj_cone(int cone, int dim, const double* v, const double* f, double* out, int64_t count,
                      hipStream_t s) {
  const int per_block = cone == 0 ? kWavesPerBlock : kBlock;
  if (count > 0)
    k_proj_cone<<<(unsigned)((count + per_block - 1) / per_block), kBlock, 0, s>>>(cone, dim, v, f, out, count);
}

void launch_pack_warm(const void* const* src, const int32_t* off, int B, int64_t maxlen, int dtype, double* out,
                      int32_t* nan_flag, hipStream_t s) {
  if (B <= 0 || maxlen <= 0) return;
  const dim3 g((unsigned)std::min<int64_t>((maxlen + 255) / 256, 1024), (unsigned)std::min(B, 4096));
  if (dtype == 0) k_pack_warm<double><<<g, 256, 0, s>>>(src, off, B, out, nan_flag);
  else k_pack_warm<float><<<g, 256, 0, s>>>(src, off, B, out, nan_flag);
}

void launch_dual_only(const KernelCtx& k, hipStream_t s, int prec) {
  if (prec == kFP32) launch_dual_t<float>(k, s, kFP32, k.it32, k.d32, k.A32, k.bpart32);
  else launch_dual_t<double>(k, s, kFP64, k.it64, k.d64, k.A64, k.bpart64);
}

}  // namespace pdcs
