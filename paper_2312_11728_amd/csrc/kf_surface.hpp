// The per-entry step of the FP64 forward and backward fits on the surface
// frame.
//
// After a propagation the covariance of a track has the surface normal as a
// null vector, so it is kept as the 5x5 covariance c[15] (packed lower
// triangle) of (a, b, ipt, phi, theta), with a, b the position along two unit
// directions of the surface:
//   barrel  a = (tx, ty, 0), the tangent (-n_y, n_x), and b = z,
//   disk    a = x, b = y.
// With E the 6x5 matrix of these directions, C = E c E^T.  In exact
// arithmetic the step is that of propagate() and update() on the 6x6
// covariance:
//   transport  c' = J c J^T with J = E'^T F E, the Jacobian between the two
//              frames; imposing the normal as a null vector is no step of its
//              own (63 multiply-adds between barrel layers instead of ~210);
//   update     S = H C H^T + V with C of rank 2 in position.  Splitting the
//              hit along the frame and the normal n, S^-1 restricted to the
//              frame is (c_pos + W)^-1 with W = V_ab - V_an V_nn^-1 V_na, the
//              residual r_ab - V_an V_nn^-1 r_n, and chi2 gains r_n^2 / V_nn:
//              a 2-D update, done as two scalar ones in the coordinates that
//              make W diagonal (~115 multiply-adds instead of ~320).  The row
//              of each measured direction is scaled by w / s instead of
//              subtracted from: where the hit is far more precise than the
//              state (z on a steep track), the difference would lose
//              log10(c / w) digits.
// The results differ from the 6x6 form's by rounding only (1e-13 on central
// tracks; chi2 agrees within 1e-8 at |eta| 5.5).  100,000
// tracks x 20 layers: 275 -> 200 us.
#pragma once

#include "kf_math.hpp"

namespace kf {

// packed index of the 5x5 covariance: 0 a, 1 b, 2 ipt, 3 phi, 4 theta
enum { SA = 0, SB = 1, SI = 2, SP = 3, ST = 4 };

template <typename T>
struct SurfState {
  T p[6];
  T c[15];
  T tx, ty;   // the direction of a (barrel), (1, 0) on a disk
  int kind;   // 0 barrel frame, 1 disk frame
  int q;
};

// Reciprocal by Newton's method from the hardware's approximation: within an
// ulp, 5 instructions instead of the division's 11.  1 / 0 gives NaN.
KF_HD inline double s_rcp(double x) {
#ifdef __HIP_DEVICE_COMPILE__
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  return fma(fma(-x, r, 1.0), r, r);
#else
  return 1.0 / x;
#endif
}

// C = E c E^T, packed 6x6
template <typename T>
KF_HD inline void expand_cov(const SurfState<T>& s, T C[21]) {
  const bool disk = s.kind == 1;
  const T* c = s.c;
  const T aa = c[sym(SA, SA)], ab = c[sym(SB, SA)], bb = c[sym(SB, SB)];
  const T ya = s.ty * aa;
  C[sym(0, 0)] = disk ? aa : s.tx * s.tx * aa;
  C[sym(1, 0)] = disk ? ab : s.tx * ya;
  C[sym(1, 1)] = disk ? bb : s.ty * ya;
  C[sym(2, 0)] = disk ? T(0) : s.tx * ab;
  C[sym(2, 1)] = disk ? T(0) : s.ty * ab;
  C[sym(2, 2)] = disk ? T(0) : bb;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const T ka = c[sym(SI + k, SA)], kb = c[sym(SI + k, SB)];
    C[sym(3 + k, 0)] = disk ? ka : s.tx * ka;
    C[sym(3 + k, 1)] = disk ? kb : s.ty * ka;
    C[sym(3 + k, 2)] = disk ? T(0) : kb;
#pragma unroll
    for (int l = 0; l <= k; ++l) C[sym(3 + k, 3 + l)] = c[sym(SI + k, SI + l)];
  }
}

// c = E^T C E of a 6x6 covariance that has the frame's normal as a null vector
template <typename T>
KF_HD inline void compress_cov(const T C[21], SurfState<T>& s) {
  const bool disk = s.kind == 1;
  T* c = s.c;
  T ca[6];   // C a
#pragma unroll
  for (int i = 0; i < 6; ++i) ca[i] = disk ? C[sym(i, 0)] : s.tx * C[sym(i, 0)] + s.ty * C[sym(i, 1)];
  c[sym(SA, SA)] = disk ? ca[0] : s.tx * ca[0] + s.ty * ca[1];
  c[sym(SB, SA)] = disk ? ca[1] : ca[2];
  c[sym(SB, SB)] = disk ? C[sym(1, 1)] : C[sym(2, 2)];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    c[sym(SI + k, SA)] = ca[3 + k];
    c[sym(SI + k, SB)] = disk ? C[sym(3 + k, 1)] : C[sym(3 + k, 2)];
#pragma unroll
    for (int l = 0; l <= k; ++l) c[sym(SI + k, SI + l)] = C[sym(3 + k, 3 + l)];
  }
}

// A covariance of full rank (after the first entry: its position is not
// confined to a surface) moved along the track onto the plane
// through the state whose normal is the transverse direction of motion:
// c = P C P^T, P the Jacobian I + g d^T of a step of length 0, d = -n /(n.g).
// The next surface's Jacobian F maps the direction of motion g to zero, so
// F P = F: the next propagation gives what it gives from C.
template <typename T>
KF_HD inline void confine_to_track_plane(const T C[21], T bz, SurfState<T>& s) {
  T sp, cp, sth, cth;
  k_sincos(s.p[4], &sp, &cp);
  k_sincos(s.p[5], &sth, &cth);
  const T cot = cth * s_rcp(sth);
  const T w = -T(s.q) * T(kCLight) * bz * s.p[3];
  s.kind = 0;
  s.tx = -sp;
  s.ty = cp;
  T M[5][6];   // P C: the rows a, b, ipt, phi, theta
#pragma unroll
  for (int j = 0; j < 6; ++j) {
    const T along = cp * C[sym(0, j)] + sp * C[sym(1, j)];
    M[0][j] = s.tx * C[sym(0, j)] + s.ty * C[sym(1, j)];
    M[1][j] = C[sym(2, j)] - cot * along;
    M[2][j] = C[sym(3, j)];
    M[3][j] = C[sym(4, j)] - w * along;
    M[4][j] = C[sym(5, j)];
  }
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    const T along = cp * M[i][0] + sp * M[i][1];
    s.c[sym(i, SA)] = s.tx * M[i][0] + s.ty * M[i][1];
    if (i >= 1) s.c[sym(i, SB)] = M[i][2] - cot * along;
    if (i >= 2) s.c[sym(i, SI)] = M[i][3];
    if (i >= 3) s.c[sym(i, SP)] = M[i][4] - w * along;
    if (i >= 4) s.c[sym(i, ST)] = M[i][5];
  }
}

// 2 atan(t) / t, series to t^12: within 6e-10 for |t| <= 0.25 (the start of a
// Newton search)
template <typename T>
KF_HD inline T two_atanc(T t) {
  const T t2 = t * t;
  T r = T(2.0 / 13.0);
  r = T(-2.0 / 11.0) + t2 * r;
  r = T(2.0 / 9.0) + t2 * r;
  r = T(-2.0 / 7.0) + t2 * r;
  r = T(2.0 / 5.0) + t2 * r;
  r = T(-2.0 / 3.0) + t2 * r;
  return T(2) + t2 * r;
}

// The point where the helix crosses the surface, with what the Jacobian needs.
template <typename T>
struct CrossPt {
  T s, x, y, z, u;    // transverse path, position, turning angle
  T sphm, cphm;       // direction there
  T dx, dy, shc;      // chord, sinc(u / 2)
};

template <typename T>
KF_HD inline void cross_eval(const T p[6], T sphi, T cphi, T cot, T w, T s, CrossPt<T>& o) {
  const T u = w * s;
  const T h = T(0.5) * u;
  T sh, ch;
  k_sincos(h, &sh, &ch);
  T shc;
  if (k_abs(h) < T(0.05)) {
    const T h2 = h * h;
    shc = T(1) - h2 * (T(1.0 / 6.0) - h2 * (T(1.0 / 120.0) - h2 * T(1.0 / 5040.0)));
  } else {
    shc = sh * s_rcp(h);
  }
  const T smid = sphi * ch + cphi * sh;
  const T cmid = cphi * ch - sphi * sh;
  const T sin_u = T(2) * sh * ch;
  const T cos_u = T(1) - T(2) * sh * sh;
  const T chord = s * shc;
  o.s = s;
  o.dx = chord * cmid;
  o.dy = chord * smid;
  o.x = p[0] + o.dx;
  o.y = p[1] + o.dy;
  o.z = p[2] + s * cot;
  o.u = u;
  o.sphm = sphi * cos_u + cphi * sin_u;
  o.cphm = cphi * cos_u - sphi * sin_u;
  o.shc = shc;
}

// First admissible crossing (the rule of crossing()).  Barrel: of the roots
// sig1 = qq / alpha and sig2 = -D / (2 qq), sig2 is taken at once where it is
// known to be the first: alpha > 0 and either qq > 0 and D < 0 (both roots
// ahead, sig2 the nearer) or qq <= -alpha (sig1 <= -1, so s1 = 2 atan(w
// sig1) / w lies more than 1 cm behind when |w| <= 1.5 and belongs to the
// turn's far end, s1 + 2 pi / |w| >= pi / |w| >= s2), and s2 > lo.  A wave
// whose tracks all do (an outgoing or incoming track between barrel layers)
// skips the second root.
template <typename T>
KF_HD inline bool cross_surface(const T p[6], T sphi, T cphi, T cot, T w, int kind, T pos, bool same,
                                CrossPt<T>& o) {
  const T lo = same ? T(kSSame) : T(-kSBack);
  if (kind == 1) {
    if (!(k_abs(cot) > T(1e-12))) return false;
    const T s = (pos - p[2]) * s_rcp(cot);
    if (!(s > lo)) return false;
    cross_eval(p, sphi, cphi, cot, w, s, o);
    o.z = pos;
    return true;
  }
  const T x = p[0], y = p[1];
  const T A = x * cphi + y * sphi;
  const T B = x * sphi - y * cphi;
  const T R2 = pos * pos;
  const T r0 = k_sqrt(x * x + y * y);
  const T D = (pos - r0) * (pos + r0);
  const T alpha = T(2) * (T(1) - w * B) - T(0.5) * w * w * D;
  const T disc = A * A + T(0.5) * alpha * D;
  if (!(disc >= T(0))) return false;
  const T sq = k_sqrt(disc);
  const T qq = -(A + k_copysign(sq, A));
  const T sig = T(-0.5) * D * s_rcp(qq);
  const T t = w * sig;
  T s = sig * two_atanc(t);
  const bool first = alpha > T(0) && (qq > T(0) ? D < T(0) : -qq >= alpha) && k_abs(w) <= T(1.5) &&
                     k_abs(t) < T(0.25) && s > lo;
  if (!first) {
    bool found = false;
    s = T(0);
    if (qq != T(0) || alpha != T(0)) {
      T s1 = path_from_sigma(qq, alpha, w);
      if (k_finite(s1)) {
        s1 = to_window(s1, lo, w);
        if (s1 > lo) {
          s = s1;
          found = true;
        }
      }
    }
    if (qq != T(0)) {
      T s2 = path_from_sigma(T(-0.5) * D, qq, w);
      if (k_finite(s2)) {
        s2 = to_window(s2, lo, w);
        if (s2 > lo && (!found || s2 < s)) {
          s = s2;
          found = true;
        }
      }
    }
    if (!found) return false;
  }
  // Newton steps on r(s)^2 - R^2, two as in crossing().  A correction ds
  // whose dropped terms, (w ds)^2 and |w| ds^2 against R, stay below a
  // hundredth of an ulp moves the point to first order (on turns of up to one
  // radian, where the series below has all its digits); one within the
  // rounding of r^2 itself, |ds| <= 2 ulp(R), ends the search.
  cross_eval(p, sphi, cphi, cot, w, s, o);
  constexpr T eps = T(2.220446e-16);
  const T tiny = T(0.01) * eps;
#pragma unroll 1
  for (int it = 0; it < 2; ++it) {
    const T f = (o.x * o.x - R2) + o.y * o.y;
    const T df = T(2) * (o.x * o.cphm + o.y * o.sphm);
    if (!(k_abs(df) > T(1e-20))) break;
    const T ds = -f * s_rcp(df);
    const T wd = w * ds;
    const T h = T(0.5) * o.u;
    if (wd * wd <= tiny && k_abs(w) * ds * ds <= tiny * pos && k_abs(h) <= T(0.5)) {
      o.s += ds;
      o.x += ds * o.cphm;
      o.y += ds * o.sphm;
      o.dx += ds * o.cphm;
      o.dy += ds * o.sphm;
      o.z += ds * cot;
      o.u += wd;
      const T sp = o.sphm, cp = o.cphm;
      o.sphm = sp + wd * cp;
      o.cphm = cp - wd * sp;
      // d sinc(h) / dh = -h / 3 (1 - h^2 / 10 + h^4 / 280 - ...), whose next
      // term, h^7 / 45360, moves less than an ulp for these h and wd
      const T h2 = h * h;
      o.shc -= T(0.5) * wd * h * (T(1.0 / 3.0) - h2 * (T(1.0 / 30.0) - h2 * T(1.0 / 840.0)));
    } else {
      cross_eval(p, sphi, cphi, cot, w, o.s + ds, o);
    }
    if (k_abs(ds) <= T(2) * eps * pos) break;
  }
  return true;
}

// sum_j r[j] x[j] + x0 over the elements that a row between barrel layers has
// (BARREL: not the columns b and theta) or over all five, term by term with
// fused multiply-adds: a zero element adds exactly nothing, so both forms
// give the same bits.
template <bool BARREL, typename T>
KF_HD inline T row_dot(const T r[5], T c0, T c1, T c2, T c3, T c4) {
  T v = r[0] * c0;
  if (!BARREL) v = k_fma(r[1], c1, v);
  v = k_fma(r[2], c2, v);
  v = k_fma(r[3], c3, v);
  if (!BARREL) v = k_fma(r[4], c4, v);
  return v;
}

// c <- J c J^T for J with rows a, b, phi given by their five elements (ja,
// jb, jp; ipt and theta unchanged).  BARREL (between barrel layers): the
// columns b and theta of rows a and phi are zero, J_bb is one.
template <bool BARREL, typename T>
KF_HD inline void transport5(T c[15], const T ja[5], const T jb[5], const T jp[5]) {
  T Ma[5], Mb[5], Mp[5];
#pragma unroll
  for (int j = 0; j < 5; ++j) {
    const T c0 = c[sym(SA, j)], c1 = c[sym(SB, j)], c2 = c[sym(SI, j)], c3 = c[sym(SP, j)], c4 = c[sym(ST, j)];
    Ma[j] = row_dot<BARREL>(ja, c0, c1, c2, c3, c4);
    Mp[j] = row_dot<BARREL>(jp, c0, c1, c2, c3, c4);
    Mb[j] = k_fma(jb[4], c4, row_dot<true>(jb, c0, c1, c2, c3, c4));
    Mb[j] = BARREL ? Mb[j] + c1 : k_fma(jb[1], c1, Mb[j]);
  }
  c[sym(SA, SA)] = row_dot<BARREL>(ja, Ma[0], Ma[1], Ma[2], Ma[3], Ma[4]);
  c[sym(SB, SA)] = row_dot<BARREL>(ja, Mb[0], Mb[1], Mb[2], Mb[3], Mb[4]);
  c[sym(SP, SA)] = row_dot<BARREL>(ja, Mp[0], Mp[1], Mp[2], Mp[3], Mp[4]);
  c[sym(SP, SP)] = row_dot<BARREL>(jp, Mp[0], Mp[1], Mp[2], Mp[3], Mp[4]);
  c[sym(SP, SB)] = row_dot<BARREL>(jp, Mb[0], Mb[1], Mb[2], Mb[3], Mb[4]);
  T bb = k_fma(jb[4], Mb[4], row_dot<true>(jb, Mb[0], Mb[1], Mb[2], Mb[3], Mb[4]));
  bb = BARREL ? bb + Mb[1] : k_fma(jb[1], Mb[1], bb);
  c[sym(SB, SB)] = bb;
  c[sym(SI, SA)] = Ma[SI];
  c[sym(SI, SB)] = Mb[SI];
  c[sym(SP, SI)] = Mp[SI];
  c[sym(ST, SA)] = Ma[ST];
  c[sym(ST, SB)] = Mb[ST];
  c[sym(ST, SP)] = Mp[ST];
}

// Highland angle squared (highland_var, without its square roots: theta0^2 is
// a product) for the inverse incidence cosine ica = 1 / |cos|, clamped at
// 1 / kGrazingCos.
template <typename T>
KF_HD inline T highland_var2(T ipt, T sth, T ica, T x_over_x0, T mass) {
  const T ps = ipt * sth;                      // 1 / p
  const T mis = mass * ps;
  const T one_m = T(1) + mis * mis;            // 1 / beta^2
  const T xl = x_over_x0 * ica;
  const T lg = T(1) + T(0.038) * k_log(xl * one_m);
  return T(0.0136 * 0.0136) * (ps * ps) * one_m * xl * (lg * lg);
}

template <typename T>
KF_HD inline void add_q5(T c[15], T ipt, T isth, T cot, T var) {
  const T ic = ipt * cot;
  c[sym(SI, SI)] += ic * ic * var;
  c[sym(ST, SI)] += -ic * var;
  c[sym(SP, SP)] += var * (isth * isth);
  c[sym(ST, ST)] += var;
}

// Propagation to the surface (kind, pos) with its material: propagate() on
// the surface frame.  Returns false, s untouched, without an admissible
// crossing.  pre is called with the state on the surface before the material.
template <typename T, typename PreMaterial = NoPreMaterial>
KF_HD inline bool propagate5(SurfState<T>& s, int kind, T pos, T x_over_x0, bool same, T bz, T mass, uint32_t& st,
                             const PreMaterial& pre = PreMaterial()) {
  const T dw = -T(s.q) * T(kCLight) * bz;
  const T w = dw * s.p[3];
  T sphi, cphi, sth, cth;
  k_sincos(s.p[4], &sphi, &cphi);
  k_sincos(s.p[5], &sth, &cth);
  const T isth = s_rcp(sth);
  const T cot = cth * isth;
  CrossPt<T> o;
  if (!cross_surface(s.p, sphi, cphi, cot, w, kind, pos, same, o)) {
    st |= TRK_NO_CROSSING;
    return false;
  }
  // partials at fixed path: ipt moves the position by (G03, G13) and the
  // direction by G43, phi moves it by (-dy, dx), theta moves z by G25
  const T f1 = u_minus_sin_over_u2(o.u);
  const T f2 = T(0.5) * o.shc * o.shc;
  const T sd = o.s * o.s * dw;
  const T G03 = sd * (o.cphm * f1 - o.sphm * f2);
  const T G13 = sd * (o.sphm * f1 + o.cphm * f2);
  const T G25 = -o.s * isth * isth;
  const T G43 = o.s * dw;
  // the new frame's directions (na_x, na_y, 0) and, on a disk, y; the path
  // moves by D.c for a displacement c, so that c maps to c + g (D.c)
  const bool disk = kind == 1, odisk = s.kind == 1;
  T ica, ntx = T(1), nty = T(0);
  bool graze;
  T ja[5], jb[5], jp[5];
  if (!disk) {
    const T rinv = s_rcp(pos);
    const T nx = o.x * rinv, ny = o.y * rinv;
    const T cn = nx * o.cphm + ny * o.sphm;   // n . g
    const T inv = -s_rcp(cn);
    const T tg = nx * o.sphm - ny * o.cphm;   // t . g
    ntx = -ny;
    nty = nx;
    // columns a (and, from a disk, b), ipt, phi of the old frame
    const T ux = odisk ? T(1) : s.tx, uy = odisk ? T(0) : s.ty;
    const T da = inv * (nx * ux + ny * uy);
    const T db = odisk ? inv * ny : T(0);
    const T di = inv * (nx * G03 + ny * G13);
    const T dp = inv * (ny * o.dx - nx * o.dy);
    ja[0] = nx * uy - ny * ux + tg * da;
    ja[1] = odisk ? nx + tg * db : T(0);
    ja[2] = nx * G13 - ny * G03 + tg * di;
    ja[3] = nx * o.dx + ny * o.dy + tg * dp;
    ja[4] = T(0);
    jb[0] = cot * da;
    jb[1] = odisk ? cot * db : T(1);
    jb[2] = cot * di;
    jb[3] = cot * dp;
    jb[4] = G25;
    jp[0] = w * da;
    jp[1] = w * db;
    jp[2] = G43 + w * di;
    jp[3] = T(1) + w * dp;
    jp[4] = T(0);
    graze = k_abs(sth * cn) < T(kGrazingCos);
    ica = k_abs(inv * isth);
  } else {
    const T inv = -s_rcp(cot);
    const T db = odisk ? T(0) : inv, dt = G25 * inv;   // only z and theta move the path
    ja[0] = odisk ? T(1) : s.tx;
    ja[1] = o.cphm * db;
    ja[2] = G03;
    ja[3] = -o.dy;
    ja[4] = o.cphm * dt;
    jb[0] = odisk ? T(0) : s.ty;
    jb[1] = odisk ? T(1) : o.sphm * db;
    jb[2] = G13;
    jb[3] = o.dx;
    jb[4] = o.sphm * dt;
    jp[0] = T(0);
    jp[1] = w * db;
    jp[2] = G43;
    jp[3] = T(1);
    jp[4] = w * dt;
    graze = k_abs(cth) < T(kGrazingCos);
    ica = k_abs(inv * isth);   // 1 / |cos theta| = |tan theta| / sin theta
  }
  // one form for the whole wave: a mixed wave would run both
  if (all_lanes(!disk && !odisk))
    transport5<true>(s.c, ja, jb, jp);
  else
    transport5<false>(s.c, ja, jb, jp);
  const T phi = s.p[4] + o.u;
  s.p[0] = o.x;
  s.p[1] = o.y;
  s.p[2] = o.z;
  s.p[4] = wrap_phi(phi);
  s.tx = ntx;
  s.ty = nty;
  s.kind = kind;
  pre(s);
  if (graze) {
    st |= TRK_GRAZING;
    ica = T(1.0 / kGrazingCos);
  }
  add_q5(s.c, s.p[3], isth, cot, highland_var2(s.p[3], sth, ica, x_over_x0, mass));
  return true;
}

// After an update of either form: the charge flip, the phi wrap.
template <typename T>
KF_HD inline void flip_and_wrap5(SurfState<T>& s, uint32_t& st) {
  if (s.p[3] < T(0)) {
    s.p[3] = -s.p[3];
    s.q = -s.q;
    s.c[sym(SI, SA)] = -s.c[sym(SI, SA)];
    s.c[sym(SI, SB)] = -s.c[sym(SI, SB)];
    s.c[sym(SP, SI)] = -s.c[sym(SP, SI)];
    s.c[sym(ST, SI)] = -s.c[sym(ST, SI)];
    st |= TRK_CHARGE_FLIP;
  }
  s.p[4] = wrap_phi(s.p[4]);
}

// Kalman update with hit m, V on the surface frame.  Returns false, nothing
// done, when V is not positive definite: update() then has to do it on the
// 6x6 covariance.
template <typename T>
KF_HD inline bool update5(SurfState<T>& s, const T m[3], const T V[6], T& chi2, uint32_t& st) {
  T r0 = m[0] - s.p[0], r1 = m[1] - s.p[1];
  const T r2 = m[2] - s.p[2];
  T* c = s.c;
  T vaa, vab, vbb, van, vbn, vnn, ra, rb, rn;
  if (s.kind == 0) {
    const T nx = s.ty, ny = -s.tx;
    const T tx0 = V[0] * s.tx + V[1] * s.ty, tx1 = V[1] * s.tx + V[2] * s.ty;
    const T nx0 = V[0] * nx + V[1] * ny, nx1 = V[1] * nx + V[2] * ny;
    vaa = s.tx * tx0 + s.ty * tx1;
    vab = V[3] * s.tx + V[4] * s.ty;
    vbb = V[5];
    van = nx * tx0 + ny * tx1;
    vbn = V[3] * nx + V[4] * ny;
    vnn = nx * nx0 + ny * nx1;
    ra = r0 * s.tx + r1 * s.ty;
    rb = r2;
    rn = r0 * nx + r1 * ny;
  } else {
    vaa = V[0];
    vab = V[1];
    vbb = V[2];
    van = V[3];
    vbn = V[4];
    vnn = V[5];
    ra = r0;
    rb = r1;
    rn = r2;
  }
  const T in = s_rcp(vnn);
  const T an = van * in, bn = vbn * in;
  const T waa = vaa - an * van, wab = vab - an * vbn, wbb = vbb - bn * vbn;
  const T det = waa * wbb - wab * wab;
  const T caa = c[sym(SA, SA)];
  if (!(vnn > T(0) && waa > T(0) && det > T(0))) return false;
  ra -= an * rn;
  rb -= bn * rn;
  // measured a with variance waa, then h = b - l a with variance wh
  const T l = wab * s_rcp(waa);
  const T wh = wbb - l * wab;
  const T is0 = s_rcp(caa + waa);
  const T z0 = ra * is0, k0 = waa * is0;
  T ca[5], ch[5];
#pragma unroll
  for (int i = 0; i < 5; ++i) ca[i] = c[sym(i, SA)];
  s.c[sym(SA, SA)] = ca[0] * k0;
#pragma unroll
  for (int i = 1; i < 5; ++i) {
    const T g = ca[i] * is0;
#pragma unroll
    for (int j = 1; j <= i; ++j) c[sym(i, j)] -= g * ca[j];
  }
#pragma unroll
  for (int i = 1; i < 5; ++i) c[sym(i, SA)] = ca[i] * k0;
  const T da0 = ca[0] * z0, db0 = ca[1] * z0;
#pragma unroll
  for (int i = 0; i < 5; ++i) ch[i] = c[sym(i, SB)] - l * c[sym(i, SA)];
  const T rh = (rb - db0) - l * (ra - da0);
  const T hh = ch[1] - l * ch[0];
  const T is1 = s_rcp(hh + wh);
  const T z1 = rh * is1, k1 = wh * is1;
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    if (i == SB) continue;
    const T g = ch[i] * is1;
#pragma unroll
    for (int j = 0; j <= i; ++j)
      if (j != SB) c[sym(i, j)] -= g * ch[j];
  }
  // row h is scaled by wh / s; then b = h + l a
#pragma unroll
  for (int i = 0; i < 5; ++i)
    if (i != SB) c[sym(i, SB)] = ch[i] * k1 + l * c[sym(i, SA)];
  c[sym(SB, SB)] = hh * k1 + l * (ch[0] * k1 + c[sym(SB, SA)]);
  chi2 = rn * rn * in + ra * z0 + rh * z1;
  const T da = da0 + ch[0] * z1, db = db0 + ch[1] * z1;
  if (s.kind == 0) {
    s.p[0] += s.tx * da;
    s.p[1] += s.ty * da;
    s.p[2] += db;
  } else {
    s.p[0] += da;
    s.p[1] += db;
  }
  s.p[3] += ca[2] * z0 + ch[2] * z1;
  s.p[4] += ca[3] * z0 + ch[3] * z1;
  s.p[5] += ca[4] * z0 + ch[4] * z1;
  flip_and_wrap5(s, st);
  const T ua = c[sym(SA, SA)], ub = c[sym(SB, SB)];
  const T tol = T(1e-3) * (ua + ub);
  if (!(c[sym(SI, SI)] > T(0)) || !(c[sym(SP, SP)] > T(0)) || !(c[sym(ST, ST)] > T(0)) || ua < -tol || ub < -tol)
    st |= TRK_COV_NOT_PSD;
  return true;
}

template <typename T>
KF_HD inline bool all_finite5(const SurfState<T>& s, T chi2) {
  bool ok = k_finite(chi2);
#pragma unroll
  for (int i = 0; i < 6; ++i) ok = ok && k_finite(s.p[i]);
#pragma unroll
  for (int i = 0; i < 15; ++i) ok = ok && k_finite(s.c[i]);
  return ok;
}

}  // namespace kf
