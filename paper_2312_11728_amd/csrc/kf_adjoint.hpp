// Hand-written reverse pass of the forward fit: the gradient of
// L = sum_t w_t chi2_t with respect to the seed states and the hit positions.
//
// The sweep runs over a track's entries from the last to the first.  The
// state entering each entry is recomputed from the nearest checkpoint written
// by the forward fit (every `seg` entries), and each entry's adjoint is the
// reverse of its three parts:
//   update     p' = p + K r, C' = C - K H C (the Joseph form has the same
//              derivative at the optimal gain), chi2 = r^T S^-1 r
//   material   C += Q(p)
//   transport  p' = g(p), C' = F(p) C F(p)^T with F = G + g_s d^T, where the
//              path length s(p) enters through the implicit-function rule
//              ds/dp = d, so the root solve itself is not differentiated.
// Symmetric-matrix adjoints are kept as symmetric full matrices (dL =
// sum_ij Cb_ij dC_ij over all 36 entries), stored packed.
#pragma once

#include "kf_track.hpp"

namespace kf {

// Gradient of <Cb, Q(p)> (Cb symmetric full-matrix adjoint, packed) with
// respect to p, added to pb, given the sines and cosines of phi and theta.
// Q as in add_q / highland_var; `seed` selects the incidence of the seed's own
// layer (radius from the position) instead of the crossing formula (radius =
// the layer radius, 1/R = rinv).  The variance is k^2 (ipt sth)^2 one_m xl
// L^2, so its logarithmic derivatives are 2 by ipt and sth and 1 + 0.076 / L
// by xl and one_m: no square root, and four reciprocals.
template <typename T>
KF_HD inline void q_grad(const T p[6], T sph, T cph, T sth, T cth, int kind, T x_over_x0, T mass, bool seed, T rinv,
                         const T cb[21], T pb[6]) {
  const T isth = k_rcp(sth);
  const T cot = cth * isth;
  const T ipt = p[3];
  const T x = p[0], y = p[1];
  const T A = cph * x + sph * y;
  T ir = rinv;
  if (seed && kind == 0) ir = k_rcp(k_sqrt(x * x + y * y));
  const T ca_raw = (kind == 0) ? sth * A * ir : cth;
  T ca = k_abs(ca_raw);
  const bool clamped = ca < T(kGrazingCos);
  if (clamped) ca = T(kGrazingCos);
  const T ica = k_rcp(ca);
  const T mis = mass * ipt * sth;
  const T one_m = T(1) + mis * mis;
  const T xl = x_over_x0 * ica;
  const T Lg = T(1) + T(0.038) * k_log(xl * one_m);
  // var = ipt v1
  const T v1 = T(0.0136 * 0.0136) * (ipt * sth * sth) * one_m * xl * (Lg * Lg);
  const T var = ipt * v1;
  const T ql = T(1) + T(0.076) * k_rcp(Lg);
  const T ic = ipt * cot;
  const T b33 = cb[sym(3, 3)], b53 = cb[sym(5, 3)], b44 = cb[sym(4, 4)], b55 = cb[sym(5, 5)];
  // Phi = b33 ic^2 var - 2 b53 ic var + b44 var isth^2 + b55 var
  const T bvar = b33 * ic * ic - T(2) * b53 * ic + b44 * isth * isth + b55;
  const T bic = T(2) * (b33 * ic - b53) * var;
  T bisth = T(2) * b44 * var * isth;
  const T bcot = bic * ipt;
  // d var / d ln ipt = d var / d ln sth = var (2 + 2 ql mis^2 / one_m)
  const T hv = bvar * (T(2) + T(2) * ql * (mis * mis) * k_rcp(one_m)) * v1;
  const T bipt = bic * cot + hv;
  T bsth = hv * ipt * isth;
  const T bca = clamped ? T(0) : -bvar * var * ql * ica;
  const T bca_raw = ca_raw < T(0) ? -bca : bca;
  T bcth = T(0), bph = T(0), bx = T(0), by = T(0);
  if (kind == 0) {
    // ca_raw = sth A ir, A = cph x + sph y; for the seed ir = 1/sqrt(x^2 + y^2)
    bsth += bca_raw * A * ir;
    const T bA = bca_raw * sth * ir;
    bx += bA * cph;
    by += bA * sph;
    bph += bA * (-sph * x + cph * y);
    if (seed) {
      const T bir = bca_raw * sth * A;
      // ir = (x^2 + y^2)^(-1/2)
      const T dr = -bir * ir * ir * ir;
      bx += dr * x;
      by += dr * y;
    }
  } else {
    bcth += bca_raw;
  }
  // cot = cth isth, isth = 1/sth
  bcth += bcot * isth;
  bisth += bcot * cth;
  bsth += -bisth * isth * isth;
  pb[0] += bx;
  pb[1] += by;
  pb[3] += bipt;
  pb[4] += bph;
  pb[5] += bsth * cth - bcth * sth;
}

// The adjoint Fb of the Jacobian F = G + g d^T, as far as it is used: at the
// non-trivial elements of G, and contracted with d and g.
template <typename T>
struct JacAdjoint {
  T b03, b04, b13, b14, b25, b43;   // Fb at these elements
  T bg[6];                          // Fb d (the rows 0, 1, 2 and 4 are used)
  T bd[6];                          // Fb^T g
};

// Contribution of <Fb, F(p, s(p))> to pb (total derivative: partials at
// fixed s plus (d/ds) * ds/dp with ds/dp = tape.d).
template <typename T>
KF_HD inline void jacobian_grad(const PropTape<T>& tp, int kind, const JacAdjoint<T>& ja, T pb[6]) {
  const HelixPt<T>& hp = tp.hp;
  const T s = tp.s, w = tp.w, dwi = tp.dw_dipt, cot = tp.cot, isth = tp.isth, sth = tp.sth, cth = tp.cth;
  const T x = hp.x, y = hp.y, sphm = hp.sphm, cphm = hp.cphm, u = hp.u, shc = hp.shc, ch = hp.ch;
  const T smid = hp.smid, cmid = hp.cmid;
  const T f1 = tp.f1, f2 = tp.f2, inv = tp.inv;
  T bG03 = ja.b03, bG04 = ja.b04, bG13 = ja.b13, bG14 = ja.b14, bG25 = ja.b25, bG43 = ja.b43;
  const T* bg = ja.bg;
  const T* bd = ja.bd;
  T bcphm = bg[0], bsphm = bg[1], bcot = bg[2], bw = bg[4];
  T bx = T(0), by = T(0), bs = T(0), bisth = T(0), bsth = T(0), bcth = T(0), bu = T(0), bdx = T(0), bdy = T(0);
  if (kind == 0) {
    const T v3 = x * tp.G03 + y * tp.G13, v4 = x * tp.G04 + y * tp.G14;
    const T binv = bd[0] * x + bd[1] * y + bd[3] * v3 + bd[4] * v4;
    const T bv0 = bd[0] * inv, bv1 = bd[1] * inv, bv3 = bd[3] * inv, bv4 = bd[4] * inv;
    bx += bv0 + bv3 * tp.G03 + bv4 * tp.G04;
    by += bv1 + bv3 * tp.G13 + bv4 * tp.G14;
    bG03 += bv3 * x;
    bG13 += bv3 * y;
    bG04 += bv4 * x;
    bG14 += bv4 * y;
    // inv = -1/den, den = x cphm + y sphm
    const T bden = binv * inv * inv;
    bx += bden * cphm;
    by += bden * sphm;
    bcphm += bden * x;
    bsphm += bden * y;
  } else {
    // d2 = inv, d5 = G25 inv, inv = -1/cot
    const T binv = bd[2] + bd[5] * tp.G25;
    bG25 += bd[5] * inv;
    bcot += binv * inv * inv;
  }
  // G03 = dxdw dwi, G13 = dydw dwi, G04 = -dy, G14 = dx, G25 = -s isth^2, G43 = s dwi
  const T bdxdw = bG03 * dwi, bdydw = bG13 * dwi;
  bdy -= bG04;
  bdx += bG14;
  bs += -bG25 * isth * isth + bG43 * dwi;
  bisth += -bG25 * T(2) * s * isth;
  // dxdw = s^2 (cphm f1 - sphm f2), dydw = s^2 (sphm f1 + cphm f2)
  const T s2 = s * s;
  bs += bdxdw * T(2) * s * (cphm * f1 - sphm * f2) + bdydw * T(2) * s * (sphm * f1 + cphm * f2);
  bcphm += bdxdw * s2 * f1 + bdydw * s2 * f2;
  bsphm += -bdxdw * s2 * f2 + bdydw * s2 * f1;
  const T bf1 = bdxdw * s2 * cphm + bdydw * s2 * sphm;
  const T bf2 = -bdxdw * s2 * sphm + bdydw * s2 * cphm;
  // f2 = shc^2 / 2; f1'(u) = f2 - 2 f1 / u
  T bshc = bf2 * shc;
  const T df1 = k_abs(u) < T(1e-3) ? T(1.0 / 6.0) - u * u * T(1.0 / 40.0) : f2 - T(2) * f1 * k_rcp(u);
  bu += bf1 * df1;
  // x = x0 + dx, y = y0 + dy
  const T bx0 = bx, by0 = by;
  bdx += bx;
  bdy += by;
  // dx = s cmid shc, dy = s smid shc
  bs += bdx * cmid * shc + bdy * smid * shc;
  const T bcmid = bdx * s * shc, bsmid = bdy * s * shc;
  bshc += bdx * s * cmid + bdy * s * smid;
  // (sphm, cphm) = sin, cos (phi0 + u); (smid, cmid) = sin, cos (phi0 + u/2)
  const T bphim = bsphm * cphm - bcphm * sphm;
  const T bphimid = bsmid * cmid - bcmid * smid;
  const T bphi0 = bphim + bphimid;
  bu += bphim;
  T bh = bphimid;
  const T h = T(0.5) * u;
  const T dsinc = k_abs(h) < T(1e-2) ? -h * T(1.0 / 3.0) + h * h * h * T(1.0 / 30.0) : (ch - shc) * k_rcp(h);
  bh += bshc * dsinc;
  bu += T(0.5) * bh;
  // u = w s, w = dwi ipt
  bw += bu * s;
  bs += bu * w;
  const T bipt = bw * dwi;
  // cot = cth isth, isth = 1/sth
  bcth += bcot * isth;
  bisth += bcot * cth;
  bsth += -bisth * isth * isth;
  const T btheta = bsth * cth - bcth * sth;
  pb[0] += bx0 + bs * tp.d[0];
  pb[1] += by0 + bs * tp.d[1];
  pb[2] += bs * tp.d[2];
  pb[3] += bipt + bs * tp.d[3];
  pb[4] += bphi0 + bs * tp.d[4];
  pb[5] += btheta + bs * tp.d[5];
}

// Reverse of the update (computed in U), given the predicted state pp, its
// covariance C (packed), the aligned hit m and V.  In: pb, Gb (packed) =
// adjoints of the updated state/covariance (after the charge flip, if it
// happened).  Out: pb, Gb = adjoints of the predicted state/covariance; mb =
// adjoint of m.  With B = C[:, 0:3], K = B S^-1, s = S^-1 r and z = K^T pb:
//   r-bar = 2 w s + z
//   S-bar = -(w s s^T + z s^T - K^T Gb K), symmetrised
//   B-bar = pb s^T - 2 Gb K
// and C-bar = Gb with S-bar and B-bar put in place, symmetrised.
template <typename U>
KF_HD inline void update_vjp(const U pp[6], const U C[21], const U m[3], const U V[6], U wchi, U pb[6], U Gb[21],
                             U mb[3]) {
  U Sp[6], Si[6];
#pragma unroll
  for (int k = 0; k < 6; ++k) Sp[k] = C[k] + V[k];
  uint32_t ist = 0;
  inverse_checked<U>(Sp, Si, ist);
  const U r[3] = {m[0] - pp[0], m[1] - pp[1], m[2] - pp[2]};
  U s[3], z[3], K[6][3], GK[6][3];
#pragma unroll
  for (int k = 0; k < 3; ++k) s[k] = Si[sym(k, 0)] * r[0] + Si[sym(k, 1)] * r[1] + Si[sym(k, 2)] * r[2];
#pragma unroll
  for (int i = 0; i < 6; ++i)
#pragma unroll
    for (int k = 0; k < 3; ++k)
      K[i][k] = C[sym(i, 0)] * Si[sym(0, k)] + C[sym(i, 1)] * Si[sym(1, k)] + C[sym(i, 2)] * Si[sym(2, k)];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    U acc = U(0);
#pragma unroll
    for (int i = 0; i < 6; ++i) acc += K[i][k] * pb[i];
    z[k] = acc;
  }
#pragma unroll
  for (int i = 0; i < 6; ++i)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      U acc = U(0);
#pragma unroll
      for (int j = 0; j < 6; ++j) acc += Gb[sym(i, j)] * K[j][k];
      GK[i][k] = acc;
    }
#pragma unroll
  for (int i = 0; i < 6; ++i)
#pragma unroll
    for (int k = 0; k <= i && k < 3; ++k) {
      U v = Gb[sym(i, k)] - GK[i][k];
      if (i < 3) {
        U n = U(0);   // (K^T Gb K)_ik
#pragma unroll
        for (int j = 0; j < 6; ++j) n += K[j][i] * GK[j][k];
        v += n - GK[k][i] - wchi * s[i] * s[k] + U(0.5) * ((pb[i] - z[i]) * s[k] + (pb[k] - z[k]) * s[i]);
      } else {
        v += U(0.5) * pb[i] * s[k];
      }
      Gb[sym(i, k)] = v;
    }
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    mb[k] = U(2) * wchi * s[k] + z[k];
    pb[k] -= mb[k];
  }
}

// Intermediates of a propagation converted to the reverse pass's type.
template <typename U, typename T>
KF_HD inline PropTape<U> tape_as(const PropTape<T>& t) {
  PropTape<U> o;
  o.s = t.s;
  o.w = t.w;
  o.dw_dipt = t.dw_dipt;
  o.sphi = t.sphi;
  o.cphi = t.cphi;
  o.sth = t.sth;
  o.cth = t.cth;
  o.isth = t.isth;
  o.cot = t.cot;
  o.f1 = t.f1;
  o.f2 = t.f2;
  o.dxdw = t.dxdw;
  o.dydw = t.dydw;
  o.G03 = t.G03;
  o.G04 = t.G04;
  o.G13 = t.G13;
  o.G14 = t.G14;
  o.G25 = t.G25;
  o.G43 = t.G43;
  o.inv = t.inv;
#pragma unroll
  for (int i = 0; i < 6; ++i) o.d[i] = t.d[i];
  o.hp.x = t.hp.x;
  o.hp.y = t.hp.y;
  o.hp.z = t.hp.z;
  o.hp.phi = t.hp.phi;
  o.hp.sphm = t.hp.sphm;
  o.hp.cphm = t.hp.cphm;
  o.hp.dx = t.hp.dx;
  o.hp.dy = t.hp.dy;
  o.hp.u = t.hp.u;
  o.hp.sh = t.hp.sh;
  o.hp.ch = t.hp.ch;
  o.hp.shc = t.hp.shc;
  o.hp.smid = t.hp.smid;
  o.hp.cmid = t.hp.cmid;
  return o;
}

// The entry that a lane of the alignment reduction loads for place e of a batch
// whose entries end before `last`, in arrays of at least one entry.  Past the
// end it is entry 0, not the batch's first: a batch of empty tracks at the end
// of the arrays has none.
KF_HD inline int64_t align_load_entry(int64_t e, int64_t last) { return e < last ? e : 0; }

// Adjoint of one entry (see the file comment).  p_in, c_in, q_in: the state
// entering the entry; q_out: the charge after the entry (it differs from q_in
// iff the update flipped it); m_raw: the hit before alignment.  pb, cb: in,
// adjoints of the state leaving the entry; out, adjoints of the state entering
// it.  hb: adjoint of the raw hit position.  The transport is retaken in the
// forward path's type T; in FP64 the forward fit takes it on the surface frame
// and rounds it differently, so that at a tangent crossing one may find a path
// where the other finds none.  Without one here the entry passes nothing back:
// hb, pb and cb are zero, and the entries before it are swept on their own.
// The reverse arithmetic runs in FP64 for both precisions: the
// covariance adjoint is of order 1/sigma^4 of the hits while the gradient
// with respect to the earlier states is of order one, so the products in the
// transport and update reverse cancel by five to six orders of magnitude,
// which FP32 cannot resolve.
template <typename T>
KF_HD inline void step_vjp(const T p_in[6], const T c_in[21], int q_in, int q_out, int j, int lay, int prev,
                           bool valid, const T m_raw[3], const T V[6], const TrackGeom<T>& g,
                           const T* __restrict__ sal, double wchi, double pb[6], double cb[21], double hb[3]) {
  using R = double;
  const int kind = g.kind[lay];
  T p[6], c[21];
#pragma unroll
  for (int i = 0; i < 6; ++i) p[i] = p_in[i];
#pragma unroll
  for (int i = 0; i < 21; ++i) c[i] = c_in[i];
  int q = q_in;
  uint32_t sst = 0;
  PropTape<T> tp;
  hb[0] = hb[1] = hb[2] = R(0);
  if (j > 0) {
    if (!propagate(p, c, q, kind, g.pos[lay], g.x0[lay], lay == prev, true, g.bz, g.mass, sst,
                   static_cast<T*>(nullptr), &tp)) {
#pragma unroll
      for (int i = 0; i < 6; ++i) pb[i] = R(0);
#pragma unroll
      for (int i = 0; i < 21; ++i) cb[i] = R(0);
      return;
    }
  } else {
    add_material_here(p, c, kind, g.x0[lay], g.mass, sst);
  }
  // p, c: the predicted state and covariance (material included)
  R P[6];
#pragma unroll
  for (int i = 0; i < 6; ++i) P[i] = p[i];
  if (valid) {
    R m[3] = {m_raw[0], m_raw[1], m_raw[2]};
    R sa = R(0), ca = R(1);
    const bool al = sal && kind == 0;
    if (al) {
      T sat, cat;
      k_sincos(sal[lay] * k_rcp(g.pos[lay]), &sat, &cat);
      sa = sat;
      ca = cat;
      m[0] = ca * R(m_raw[0]) - sa * R(m_raw[1]);
      m[1] = sa * R(m_raw[0]) + ca * R(m_raw[1]);
      m[2] = R(m_raw[2]) + R(sal[kMaxLayers + lay]);
    }
    if (q_out != q) {
      // the update flipped the charge: ipt, q and row/column 3 changed sign
      pb[3] = -pb[3];
#pragma unroll
      for (int i = 0; i < 6; ++i)
        if (i != 3) cb[sym(3, i)] = -cb[sym(3, i)];
    }
    R C[21], Vd[6], mb[3];
#pragma unroll
    for (int i = 0; i < 21; ++i) C[i] = c[i];
#pragma unroll
    for (int i = 0; i < 6; ++i) Vd[i] = V[i];
    update_vjp<R>(P, C, m, Vd, wchi, pb, cb, mb);
    // m = R(a) h (barrel alignment): h-bar = R^T m-bar
    hb[0] = ca * mb[0] + sa * mb[1];
    hb[1] = -sa * mb[0] + ca * mb[1];
    hb[2] = mb[2];
  }
  // material: C_pred = C_prop + Q(p_pred)
  if (j > 0) {
    const PropTape<R> td = tape_as<R>(tp);
    R sph = td.hp.sphm, cph = td.hp.cphm, sth = td.sth, cth = td.cth;
    if constexpr (sizeof(T) == 4) {   // to the digits of R, not of the tape
      k_sincos(P[4], &sph, &cph);
      k_sincos(P[5], &sth, &cth);
    }
    q_grad<R>(P, sph, cph, sth, cth, kind, R(g.x0[lay]), R(g.mass), false, k_rcp(R(g.pos[lay])), cb, pb);
    // Transport: p = g(p_in), C_prop = F C_in F^T, F = G + g d^T.  With Gb the
    // adjoint of C_prop and GF = Gb F = Gb G + (Gb g) d^T:
    //   C-bar_in = F^T GF = G^T GF + d e^T, e = GF^T g
    //   F-bar = 2 GF C_in, at the elements of G and as F-bar d = 2 GF (C_in d)
    //   and F-bar^T g = 2 C_in e
    const R gv[6] = {td.hp.cphm, td.hp.sphm, td.cot, R(0), td.w, R(0)};
    const R* d = td.d;
    R GF[6][6];
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      const R b0 = cb[sym(i, 0)], b1 = cb[sym(i, 1)], b2 = cb[sym(i, 2)], b3 = cb[sym(i, 3)], b4 = cb[sym(i, 4)],
              b5 = cb[sym(i, 5)];
      const R u = b0 * gv[0] + b1 * gv[1] + b2 * gv[2] + b4 * gv[4];   // (Gb g)_i
      GF[i][0] = b0 + u * d[0];
      GF[i][1] = b1 + u * d[1];
      GF[i][2] = b2 + u * d[2];
      GF[i][3] = b3 + td.G03 * b0 + td.G13 * b1 + td.G43 * b4 + u * d[3];
      GF[i][4] = b4 + td.G04 * b0 + td.G14 * b1 + u * d[4];
      GF[i][5] = b5 + td.G25 * b2 + u * d[5];
    }
    R e[6];
#pragma unroll
    for (int b = 0; b < 6; ++b) e[b] = gv[0] * GF[0][b] + gv[1] * GF[1][b] + gv[2] * GF[2][b] + gv[4] * GF[4][b];
#pragma unroll
    for (int b = 0; b < 6; ++b)
#pragma unroll
      for (int a = b; a < 6; ++a) {
        R v = GF[a][b] + d[a] * e[b];
        if (a == 3) v += td.G03 * GF[0][b] + td.G13 * GF[1][b] + td.G43 * GF[4][b];
        if (a == 4) v += td.G04 * GF[0][b] + td.G14 * GF[1][b];
        if (a == 5) v += td.G25 * GF[2][b];
        cb[sym(a, b)] = v;
      }
    JacAdjoint<R> ja;
    auto fb = [&](int a, int b) {   // F-bar at (a, b)
      R acc = R(0);
#pragma unroll
      for (int k = 0; k < 6; ++k) acc += GF[a][k] * R(c_in[sym(k, b)]);
      return R(2) * acc;
    };
    ja.b03 = fb(0, 3);
    ja.b04 = fb(0, 4);
    ja.b13 = fb(1, 3);
    ja.b14 = fb(1, 4);
    ja.b25 = fb(2, 5);
    ja.b43 = fb(4, 3);
    R cd[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      R v = R(0), h = R(0);
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        v += R(c_in[sym(i, k)]) * d[k];
        h += R(c_in[sym(i, k)]) * e[k];
      }
      cd[i] = v;
      ja.bd[i] = R(2) * h;
    }
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      R v = R(0);
#pragma unroll
      for (int k = 0; k < 6; ++k) v += GF[i][k] * cd[k];
      ja.bg[i] = R(2) * v;
    }
    // p-bar_in = F^T p-bar + d<F-bar, F>/dp
    const R gp = gv[0] * pb[0] + gv[1] * pb[1] + gv[2] * pb[2] + gv[4] * pb[4];
    R pbi[6];
    pbi[0] = pb[0] + gp * d[0];
    pbi[1] = pb[1] + gp * d[1];
    pbi[2] = pb[2] + gp * d[2];
    pbi[3] = pb[3] + td.G03 * pb[0] + td.G13 * pb[1] + td.G43 * pb[4] + gp * d[3];
    pbi[4] = pb[4] + td.G04 * pb[0] + td.G14 * pb[1] + gp * d[4];
    pbi[5] = pb[5] + td.G25 * pb[2] + gp * d[5];
    jacobian_grad(td, kind, ja, pbi);
#pragma unroll
    for (int i = 0; i < 6; ++i) pb[i] = pbi[i];
  } else {
    // the seed's own layer: C = C_in + Q(p_in), p unchanged
    R Pin[6], sph, cph, sth, cth;
#pragma unroll
    for (int i = 0; i < 6; ++i) Pin[i] = p_in[i];
    k_sincos(Pin[4], &sph, &cph);
    k_sincos(Pin[5], &sth, &cth);
    q_grad<R>(Pin, sph, cph, sth, cth, kind, R(g.x0[lay]), R(g.mass), true, R(0), cb, pb);
  }
}

// State entering entry j (relative to the first valid entry k0) of track t:
// the seed for j = 0, else the checkpoint before entry 1 + m seg followed by
// the entries up to j - 1.  Also returns the layer of entry j - 1 (prev).
template <typename T, typename Acc>
KF_HD inline void state_before(const AdjArgs<T>& a, const TrackGeom<T>& g, const T* __restrict__ sal, int64_t t,
                               const Acc& acc, int k0, int j, T p[6], T c[21], int& q, int& prev) {
  const FitArgs<T>& f = a.f;
  const int64_t ld = f.ld;
  int jstart;
  if (j == 0) {
#pragma unroll
    for (int i = 0; i < 6; ++i) p[i] = f.seed_state[i * ld + t];
#pragma unroll
    for (int i = 0; i < 21; ++i) c[i] = f.seed_cov[i * ld + t];
    q = f.seed_charge[t];
    jstart = 0;
  } else {
    const int64_t cst = ld * int64_t(f.n_seg);
    const int mslot = (j - 1) / f.seg;
    const T* base = f.ckpt + int64_t(mslot) * ld + t;
#pragma unroll
    for (int i = 0; i < 6; ++i) p[i] = base[i * cst];
#pragma unroll
    for (int i = 0; i < 21; ++i) c[i] = base[(6 + i) * cst];
    q = int(base[27 * cst]);
    jstart = 1 + mslot * f.seg;
  }
  int lay;
  bool valid;
  T m[3], V[6];
  acc.load(k0 + (jstart > 0 ? jstart - 1 : 0), lay, valid, m, V);
  prev = lay;
  for (int jj = jstart; jj < j; ++jj) {
    acc.load(k0 + jj, lay, valid, m, V);
    T c2;
    uint32_t sst = 0;
    step_forward(p, c, q, jj, lay, prev, valid, m, V, g, sal, c2, sst);
    prev = lay;
  }
}

// A bad layer id stops the forward fit.  The refill, which does not know where
// a fit stopped, leaves the state as it is there: no later one is read.
template <typename T>
KF_HD inline bool known_layer(const TrackGeom<T>& g, int lay) {
  return lay >= 0 && lay < g.n_layers;
}

// With a state buffer: the states before entries js .. jhi (relative to the
// first valid entry k0, 1 <= js <= jhi) of track t, recomputed from the
// checkpoint of their segment in one pass and stored in slots js - 1 ..
// jhi - 1 ([slot][kSegVals][n]).
template <typename T, typename Acc>
KF_HD inline void fill_segment(const AdjArgs<T>& a, const TrackGeom<T>& g, const T* __restrict__ sal, int64_t t,
                               const Acc& acc, int k0, int js, int jhi) {
  const int64_t n = a.f.n;
  T p[6], c[21];
  int q, prev;
  state_before(a, g, sal, t, acc, k0, js, p, c, q, prev);
  for (int j = js;; ++j) {
    T* slot = a.seg_buf + int64_t(j - 1) * kSegVals * n + t;
#pragma unroll
    for (int i = 0; i < 6; ++i) slot[i * n] = p[i];
#pragma unroll
    for (int i = 0; i < 21; ++i) slot[(6 + i) * n] = c[i];
    slot[27 * n] = T(q);
    if (j == jhi) break;
    int lay;
    bool valid;
    T m[3], V[6];
    acc.load(k0 + j, lay, valid, m, V);
    if (known_layer(g, lay)) {
      T c2;
      uint32_t sst = 0;
      step_forward(p, c, q, j, lay, prev, valid, m, V, g, sal, c2, sst);
    }
    prev = lay;
  }
}

// The states before entries 1 .. n_steps - 1 of track t (len entries) for
// the reverse pass, segment by segment, each from its own checkpoint: the
// same forward steps the reverse pass would take to reach each of them.
// This is the per-track form (host builds); the device kernel takes the same
// steps with the wave's hits staged through LDS.
template <typename T, typename Acc>
KF_HD inline void refill_track(const AdjArgs<T>& a, const TrackGeom<T>& g, const T* __restrict__ sal, int64_t t,
                               const Acc& acc, int len) {
  const FitArgs<T>& f = a.f;
  if (len > f.max_len) len = f.max_len;
  int k0 = 0;
  while (k0 < len && !acc.valid(k0)) ++k0;
  const int n_steps = len - k0;
  for (int js = 1; js < n_steps; js += f.seg) {
    const int jhi = js + f.seg - 1 < n_steps - 1 ? js + f.seg - 1 : n_steps - 1;
    fill_segment(a, g, sal, t, acc, k0, js, jhi);
  }
}

// Entries, counted from the first valid one, that the forward fit completed
// on a track it stopped or flagged (a failed crossing, a non-finite step, a
// bad layer id, or an input it cut short): its steps taken again from the
// seed, in the fit's own form.  The 6x6 form of step_vjp() may round a tangent
// crossing to the other side in FP64 and count an entry whose states the fit
// never wrote.  Any other track completed all of them.
template <typename T, typename Acc>
KF_HD inline int steps_done(const AdjArgs<T>& a, const TrackGeom<T>& g, const T* __restrict__ sal, int64_t t,
                            const Acc& acc, int k0, int n_steps) {
  FitArgs<T> fa = a.f;
  fa.ckpt = nullptr;   // read here, not written again
  FitState<T> f;
  T bk[28];
  begin_fit(fa, t, g.bz, f, bk, 1);
  for (int j = 0; j < n_steps; ++j) {
    int lay;
    bool valid;
    T m[3], V[6];
    acc.load(k0 + j, lay, valid, m, V);
    if (!fit_entry<false, kFuseAny>(fa, g, sal, t, j, lay, valid, m, V, f, bk, 1)) return j;
  }
  return n_steps;
}

// Whether the forward fit's status says that it may not have completed the track.
template <typename T>
KF_HD inline bool was_stopped(const AdjArgs<T>& a, int64_t t) {
  return a.fwd_status && (a.fwd_status[t] & (TRK_NO_CROSSING | TRK_NONFINITE | TRK_BAD_INPUT));
}

// The entries of track t (len of them) that a fit uses: k0 the first valid
// one, n_steps from there.
template <typename Acc>
KF_HD inline void fitted_range(const Acc& acc, int len, int max_len, int& k0, int& n_steps) {
  if (len > max_len) len = max_len;
  k0 = 0;
  while (k0 < len && !acc.valid(k0)) ++k0;
  n_steps = len - k0;
}

// The states of track t where every one is stored: that entering entry j is in
// slot j - 1 of the buffer the refill pass wrote, or (seg = 1) of the
// checkpoints; for j = 0 it is the seed.
template <typename T>
struct StoredStates {
  const FitArgs<T>& f;
  const int64_t t, st, slot_st;
  const T* const slots;
  KF_HD inline StoredStates(const AdjArgs<T>& a, int64_t track)
      : f(a.f),
        t(track),
        st(a.seg_buf ? a.f.n : a.f.ld * int64_t(a.f.n_seg)),
        slot_st(a.seg_buf ? kSegVals * a.f.n : a.f.ld),
        slots((a.seg_buf ? a.seg_buf : a.f.ckpt) + track) {}
  KF_HD inline void before(int j, T p[6], T c[21], int& q) const {   // j >= 1
    const T* slot = slots + int64_t(j - 1) * slot_st;
#pragma unroll
    for (int i = 0; i < 6; ++i) p[i] = slot[i * st];
#pragma unroll
    for (int i = 0; i < 21; ++i) c[i] = slot[(6 + i) * st];
    q = int(slot[27 * st]);
  }
  KF_HD inline void seed(T p[6], T c[21], int& q) const {
#pragma unroll
    for (int i = 0; i < 6; ++i) p[i] = f.seed_state[i * f.ld + t];
#pragma unroll
    for (int i = 0; i < 21; ++i) c[i] = f.seed_cov[i * f.ld + t];
    q = f.seed_charge[t];
  }
};

// Reverse sweep over the n_done entries that the forward fit completed of
// track t (len entries, the first at e0 of the hit arrays), read through
// `acc`.  STORED: the state before every entry is read (StoredStates); else it
// is recomputed from its segment's checkpoint.  The stored form is for host
// builds: the device kernel takes the same steps on the same states with the
// wave's hits and their gradients going through LDS.  The charge after the last
// completed entry is not needed: the adjoints that a flip there would change
// sign of are zero.
template <bool STORED, typename T, typename Acc>
KF_HD inline void adjoint_sweep(const AdjArgs<T>& a, const TrackGeom<T>& g, const T* __restrict__ sal, int64_t t,
                                const Acc& acc, int len, int64_t e0, int k0, int n_done) {
  const FitArgs<T>& f = a.f;
  const int64_t ld = f.ld, nh = f.n_hits;
  const auto hit_grad = [&](int k, const double* h) {
    const int64_t e = e0 + k;
    a.grad_hit[e] = T(h[0]);
    a.grad_hit[nh + e] = T(h[1]);
    a.grad_hit[2 * nh + e] = T(h[2]);
  };
  // entries outside the fit: before the first valid one, past max_len or the
  // track's stop
  const double none[3] = {0.0, 0.0, 0.0};
  for (int k = 0; k < k0 && k < len; ++k) hit_grad(k, none);
  for (int k = k0 + n_done; k < len; ++k) hit_grad(k, none);
  const double wchi = a.w ? double(a.w[t]) : 1.0;
  double pb[6], cb[21];
#pragma unroll
  for (int i = 0; i < 6; ++i) pb[i] = 0.0;
#pragma unroll
  for (int i = 0; i < 21; ++i) cb[i] = 0.0;
  int q_after = 0;
  bool last = true;
  const StoredStates<T> stored(a, t);
  for (int j = n_done - 1; j >= 0; --j) {
    T p[6], c[21];
    int q, prev;
    int lay;
    bool valid;
    T m[3], V[6];
    acc.load(k0 + j, lay, valid, m, V);
    if constexpr (STORED) {
      if (j >= 1) {
        stored.before(j, p, c, q);
        prev = acc.layer(k0 + j - 1);
      } else {
        stored.seed(p, c, q);
        prev = lay;
      }
    } else {
      state_before(a, g, sal, t, acc, k0, j, p, c, q, prev);
      if (j == 0) prev = lay;
    }
    double hb[3];
    step_vjp(p, c, q, last ? q : q_after, j, lay, prev, valid, m, V, g, sal, wchi, pb, cb, hb);
    hit_grad(k0 + j, hb);   // zero for a hole
    q_after = q;
    last = false;
  }
#pragma unroll
  for (int i = 0; i < 6; ++i) a.grad_seed[i * ld + t] = T(pb[i]);
}

// Reverse pass of track t, for host builds: what the device's stop kernel and
// its sweep do to the track.
template <typename T, typename Acc>
KF_HD inline void adjoint_track(const AdjArgs<T>& a, const TrackGeom<T>& g, const T* __restrict__ sal, int64_t t,
                                const Acc& acc, int len, int64_t e0) {
  int k0, n;
  fitted_range(acc, len, a.f.max_len, k0, n);
  if (n > 0 && was_stopped(a, t)) n = steps_done(a, g, sal, t, acc, k0, n);
  if (a.seg_buf || a.f.seg == 1)
    adjoint_sweep<true>(a, g, sal, t, acc, len, e0, k0, n);
  else
    adjoint_sweep<false>(a, g, sal, t, acc, len, e0, k0, n);
}

}  // namespace kf
