// Host check of the two FP64 crossings, crossing() of the 6x6 step and
// cross_surface() of the surface frame, over random states and cylinders, half
// of them close to the largest radius that the helix reaches: both find a
// crossing or neither does, at the same path, and the half-angle sinc that the
// Jacobian takes is that of the turning angle.
#include <cmath>
#include <cstdio>
#include <random>

#include "kf_surface.hpp"

int main() {
  std::mt19937_64 rng(17);
  std::uniform_real_distribution<double> u(0.0, 1.0);
  long found = 0, differ = 0, apart = 0, sinc_off = 0;
  double worst = 0.0;
  for (long i = 0; i < 2000000; ++i) {
    const double r = 200.0 * u(rng), psi = 6.283185307 * u(rng), phi = 6.283185307 * u(rng);
    const double w = (u(rng) < 0.5 ? -1 : 1) * std::exp(std::log(1e-4) + u(rng) * std::log(1e4));
    const double p[6] = {r * std::cos(psi), r * std::sin(psi), 3.0, 1.0, phi, 1.2};
    const double sphi = std::sin(phi), cphi = std::cos(phi), cot = 1.0 / std::tan(1.2);
    // the helix's circle about (x - sphi / w, y + cphi / w)
    const double rho = 1.0 / std::fabs(w), far = std::hypot(p[0] - sphi / w, p[1] + cphi / w) + rho;
    double R = std::exp(u(rng) * std::log(300.0));
    if (u(rng) < 0.5) R = far * (1.0 - std::pow(10.0, -1.0 - 13.0 * u(rng)));
    const bool same = u(rng) < 0.2;
    double s;
    kf::HelixPt<double> hp;
    kf::CrossPt<double> o;
    const bool six = kf::crossing<kf::kFuseAny>(p, sphi, cphi, cot, w, 0, R, same, s, hp);
    const bool five = kf::cross_surface(p, sphi, cphi, cot, w, 0, R, same, o);
    if (six != five) {
      if (++differ < 5) std::printf("r %.17g psi %.17g phi %.17g w %.17g R %.17g: %d %d\n", r, psi, phi, w, R, six, five);
      continue;
    }
    if (!six) continue;
    ++found;
    if (!(std::fabs(s - o.s) <= 1e-6 * R)) ++apart;
    for (const double* x : {&hp.u, &o.u}) {
      const double shc = x == &hp.u ? hp.shc : o.shc;
      const long double h = 0.5L * *x;
      const double err = double(fabsl(shc - (h == 0.0L ? 1.0L : sinl(h) / h)));
      worst = std::fmax(worst, err);
      if (!(err <= 8.9e-16)) ++sinc_off;   // 4 units in the last place of 1
    }
  }
  std::printf("found %ld, by one only %ld, apart %ld, sinc off %ld (worst %.3g)\n", found, differ, apart, sinc_off, worst);
  return differ || apart || sinc_off || found < 500000;
}
