// Host checks of the reverse sweep at a crossing that the forward fit and the
// sweep may judge differently.
//   step  step_vjp() of a step whose surface is out of reach passes zeros back.
//   done  steps_done() counts the entries that the forward fit completed, for
//         layers whose radius lies between those that the fit's state and the
//         6x6 step's state of the same track reach.
//   layer the refill of a track with a bad layer id reads no layer that is not
//         there (under the address sanitizer).
#include <cmath>
#include <cstdio>
#include <cstring>
#include <random>
#include <vector>

#include "kf_adjoint.hpp"

namespace {

constexpr double kMass = 0.13957, kBz = 3.8;

template <typename T>
int unreachable_step() {
  const int32_t kind[2] = {0, 1};
  const T pos[2] = {T(300), T(-5)}, x0[2] = {T(0.02), T(0.02)};
  const kf::TrackGeom<T> g{kind, pos, x0, 2, T(kBz), T(kMass)};
  // 1/pT = 2 on a helix that never reaches 300 cm, nor z = -5 cm going up
  const T p[6] = {T(4), T(0), T(1), T(2), T(0.1), T(1.2)};
  T c[21] = {};
  for (int i = 0; i < 6; ++i) c[kf::sym(i, i)] = T(1e-4);
  const T m[3] = {T(10), T(1), T(2)}, V[6] = {T(1e-4), T(0), T(1e-4), T(0), T(0), T(1e-4)};
  int bad = 0;
  for (int lay = 0; lay < 2; ++lay)
    for (int valid = 0; valid < 2; ++valid) {
      double pb[6], cb[21], hb[3] = {1.0, 1.0, 1.0};
      for (double& v : pb) v = 1.0;
      for (double& v : cb) v = 1.0;
      kf::step_vjp(p, c, 1, 1, 3, lay, -1, valid != 0, m, V, g, static_cast<const T*>(nullptr), 1.0, pb, cb, hb);
      for (double v : pb) bad += !(v == 0.0);
      for (double v : cb) bad += !(v == 0.0);
      for (double v : hb) bad += !(v == 0.0);
    }
  std::printf("step: %d values not zero\n", bad);
  return bad != 0;
}

// The largest radius that a state reaches by the rule of crossing() (SIX) or
// cross_surface(), by bisection to the last digit.
template <bool SIX>
double reach(const double p[6], int q) {
  const double w = -q * kf::kCLight * kBz * p[3], cot = 1.0 / std::tan(p[5]);
  const double sphi = std::sin(p[4]), cphi = std::cos(p[4]);
  double lo = std::hypot(p[0], p[1]) + 1.0, hi = 1000.0;
  for (int i = 0; i < 200; ++i) {
    const double mid = 0.5 * (lo + hi);
    bool ok;
    if (SIX) {
      double s;
      kf::HelixPt<double> hp;
      ok = kf::crossing<kf::kFuseAny>(p, sphi, cphi, cot, w, 0, mid, false, s, hp);
    } else {
      kf::CrossPt<double> o;
      ok = kf::cross_surface(p, sphi, cphi, cot, w, 0, mid, false, o);
    }
    (ok ? lo : hi) = mid;
  }
  return lo;
}

int completed_entries() {
  constexpr int n_hit = 5, n_lay = n_hit + 2;
  std::mt19937_64 rng(3);
  std::uniform_real_distribution<double> u(0.0, 1.0);
  std::normal_distribution<double> gauss;
  long edge = 0, bad = 0;
  for (int trial = 0; trial < 4000; ++trial) {
    // a track from the beam line that turns back between 40 and 60 cm
    int32_t kind[n_lay] = {};
    double pos[n_lay] = {4, 8, 12, 16, 20, 0, 0}, x0[n_lay];
    for (double& x : x0) x = 0.02;
    const kf::TrackGeom<double> g{kind, pos, x0, n_lay, kBz, kMass};
    const int q = u(rng) < 0.5 ? -1 : 1;
    const double rho = 20.0 + 10.0 * u(rng), ipt = 1.0 / (kf::kCLight * kBz * rho), cot = 2.0 * u(rng) - 1.0;
    const double w = -q * kf::kCLight * kBz * ipt, origin[6] = {0, 0, 0, ipt, 0.3, std::atan2(1.0, cot)};
    double hit[3][n_lay], V[6][n_lay], seed[6], sc[21] = {};
    int16_t layer[n_lay];
    uint8_t valid[n_lay];
    for (int k = 0; k < n_lay; ++k) {
      kf::HelixPt<double> hp;
      double s;
      const double R = k < n_hit ? pos[k] : 2.0 * rho;
      kf::crossing<kf::kFuseAny>(origin, std::sin(0.3), std::cos(0.3), cot, w, 0, std::fmin(R, 1.99 * rho), false, s, hp);
      hit[0][k] = hp.x + 0.002 * gauss(rng);
      hit[1][k] = hp.y + 0.002 * gauss(rng);
      hit[2][k] = hp.z + 0.002 * gauss(rng);
      for (int i = 0; i < 6; ++i) V[i][k] = 0.0;
      V[0][k] = V[2][k] = V[5][k] = 4e-6;
      layer[k] = int16_t(k);
      valid[k] = 1;
      if (k == 0) {
        const double at[6] = {hp.x, hp.y, hp.z, ipt, hp.phi, origin[5]};
        for (int i = 0; i < 6; ++i) seed[i] = at[i];
      }
    }
    const double sd[6] = {0.01, 0.01, 0.01, 0.1, 0.02, 0.02};
    for (int i = 0; i < 6; ++i) sc[kf::sym(i, i)] = sd[i] * sd[i];
    const int8_t sq = int8_t(q);
    const int32_t off[2] = {0, n_lay};
    double state[6], cov[21], chi2, ckpt[28 * (n_lay - 1)];
    int8_t qo;
    int32_t ndf;
    uint32_t status;
    const auto fit = [&](int max_len) {
      kf::FitArgs<double> a{};
      a.n = a.ld = 1;
      a.n_hits = n_lay;
      a.max_len = max_len;
      a.seed_state = seed;
      a.seed_cov = sc;
      a.seed_charge = &sq;
      a.hit_offsets = off;
      a.hit_layer = layer;
      a.hit_valid = valid;
      a.hit_pos = &hit[0][0];
      a.hit_cov = &V[0][0];
      a.state_out = state;
      a.cov_out = cov;
      a.charge_out = &qo;
      a.chi2 = &chi2;
      a.ndf = &ndf;
      a.ckpt = ckpt;
      a.seg = 1;
      a.n_seg = n_lay - 1;
      a.trk_status = &status;
      status = 0;
      double bk[28];
      kf::fit_slot<double, 0>(a, g, static_cast<const double*>(nullptr), 0, bk, 1);
      return a;
    };
    // the state after the hits, in the fit's form and by 6x6 steps
    fit(n_hit);
    const int ndf_hits = ndf;
    double p6[6], c6[21];
    int q6 = q;
    for (int i = 0; i < 6; ++i) p6[i] = seed[i];
    for (int i = 0; i < 21; ++i) c6[i] = sc[i];
    for (int k = 0; k < n_hit; ++k) {
      double m[3], v[6], c2;
      for (int i = 0; i < 3; ++i) m[i] = hit[i][k];
      for (int i = 0; i < 6; ++i) v[i] = V[i][k];
      uint32_t st = 0;
      kf::step_forward(p6, c6, q6, k, k, k > 0 ? k - 1 : k, true, m, v, g, static_cast<const double*>(nullptr), c2, st);
    }
    const double r5 = reach<false>(state, qo), r6 = reach<true>(p6, q6);
    const double between = 0.5 * (r5 + r6);
    if (!(between > r5 && between < r6)) continue;   // the fit stops, the 6x6 step would not
    pos[n_hit] = between;
    pos[n_hit + 1] = 20.0;
    const kf::FitArgs<double> a = fit(n_lay);
    if (!(status & kf::TRK_NO_CROSSING) || ndf != ndf_hits) continue;
    ++edge;
    kf::AdjArgs<double> r{};
    r.f = a;
    r.fwd_status = &status;
    const kf::CsrTrack<double> acc{r.f, 0};
    bad += kf::steps_done(r, g, static_cast<const double*>(nullptr), 0, acc, 0, n_lay) != n_hit;
  }
  std::printf("done: %ld stopped on the edge, %ld counted otherwise\n", edge, bad);
  return bad || edge < 100;
}

int bad_layer() {
  constexpr int n_lay = 6, n_ent = 8, seg = 3, n_seg = (n_ent - 1 + seg - 1) / seg;
  const std::vector<int32_t> kind(n_lay, 0);
  const std::vector<double> pos{4, 8, 12, 16, 20, 24}, x0(n_lay, 0.02);
  const kf::TrackGeom<double> g{kind.data(), pos.data(), x0.data(), n_lay, kBz, kMass};
  const double seed[6] = {4, 0, 1, 0.5, 0.1, 1.2};
  double sc[21] = {};
  for (int i = 0; i < 6; ++i) sc[kf::sym(i, i)] = 1e-4;
  const int8_t q = 1;
  const int32_t off[2] = {0, n_ent};
  for (int bad : {-1, n_lay}) {
    std::vector<int16_t> layer{0, 1, 2, 3, 4, int16_t(bad), 5, 5};
    std::vector<uint8_t> valid(n_ent, 1);
    std::vector<double> hit(3 * n_ent), V(6 * n_ent, 0.0), ckpt(28 * n_seg), buf(size_t(n_ent - 1) * kf::kSegVals);
    for (int k = 0; k < n_ent; ++k) {
      hit[k] = 4.0 + 4.0 * k;
      hit[n_ent + k] = 0.1 * k;
      hit[2 * n_ent + k] = 1.0 + k;
      V[k] = V[2 * n_ent + k] = V[5 * n_ent + k] = 1e-4;
    }
    for (int s = 0; s < n_seg; ++s) {   // any states will do
      for (int i = 0; i < 6; ++i) ckpt[i * n_seg + s] = seed[i];
      for (int i = 0; i < 21; ++i) ckpt[(6 + i) * n_seg + s] = sc[i];
      ckpt[27 * n_seg + s] = 1.0;
    }
    kf::AdjArgs<double> r{};
    r.f.n = r.f.ld = 1;
    r.f.n_hits = n_ent;
    r.f.max_len = n_ent;
    r.f.seed_state = seed;
    r.f.seed_cov = sc;
    r.f.seed_charge = &q;
    r.f.hit_offsets = off;
    r.f.hit_layer = layer.data();
    r.f.hit_valid = valid.data();
    r.f.hit_pos = hit.data();
    r.f.hit_cov = V.data();
    r.f.ckpt = ckpt.data();
    r.f.seg = seg;
    r.f.n_seg = n_seg;
    r.seg_buf = buf.data();
    const kf::CsrTrack<double> acc{r.f, 0};
    kf::refill_track(r, g, static_cast<const double*>(nullptr), 0, acc, n_ent);
  }
  std::printf("layer: read\n");
  return 0;
}

}  // namespace

int main(int argc, char** argv) {
  if (argc == 2 && !std::strcmp(argv[1], "step")) return unreachable_step<float>() | unreachable_step<double>();
  if (argc == 2 && !std::strcmp(argv[1], "done")) return completed_entries();
  if (argc == 2 && !std::strcmp(argv[1], "layer")) return bad_layer();
  return 2;
}
