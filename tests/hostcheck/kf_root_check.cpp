// Host check of the barrel crossing's shortcut: wherever near_root() answers,
// first_root() (the full rule) gives the same bits.  Random quadratics of
// states inside, on and outside the cylinder, moving outwards, inwards and
// along it, with curvatures from 0 to 2 / cm and both lower ends of the path.
#include <cmath>
#include <cstdio>
#include <random>

#include "kf_math.hpp"

template <typename T>
int check(const char* name) {
  std::mt19937_64 rng(11);
  std::uniform_real_distribution<double> u(0.0, 1.0);
  long taken = 0, outward = 0, inward = 0, bad = 0;
  const long total = 2000000;
  for (long i = 0; i < total; ++i) {
    const T R = T(std::exp(std::log(1.0) + u(rng) * std::log(200.0)));
    // radius: anywhere, or within a few units in the last place of R
    const int where = int(u(rng) * 4);
    const double f = where == 0 ? u(rng) * 2 : where == 1 ? u(rng) : where == 2 ? 1.0 + 1e-6 * (u(rng) - 0.5) : 1.0 + 0.02 * (u(rng) - 0.5);
    const double r = double(R) * f, psi = u(rng) * 6.283185307, al = (u(rng) < 0.7 ? 0.6 : 3.2) * (2 * u(rng) - 1) + (u(rng) < 0.5 ? 0.0 : 3.14159265);
    const T x = T(r * std::cos(psi)), y = T(r * std::sin(psi));
    const T cphi = T(std::cos(psi + al)), sphi = T(std::sin(psi + al));
    const T w = u(rng) < 0.02 ? T(0) : T((u(rng) < 0.5 ? -1 : 1) * std::exp(std::log(1e-6) + u(rng) * std::log(2e6)));
    const T lo = u(rng) < 0.2 ? T(kf::kSSame) : T(-kf::kSBack);
    const T A = x * cphi + y * sphi, B = x * sphi - y * cphi;
    const T r0 = std::sqrt(x * x + y * y);
    const T D = (R - r0) * (R + r0);
    const T alpha = T(2) * (T(1) - w * B) - T(0.5) * w * w * D;
    const T disc = A * A + T(0.5) * alpha * D;
    if (!(disc >= T(0))) continue;
    const T qq = -(A + std::copysign(std::sqrt(disc), A));
    T near = T(0), full = T(0);
    if (!kf::near_root(qq, alpha, D, w, lo, near)) continue;
    ++taken;
    (A > T(0) ? outward : inward) += 1;
    if (!kf::first_root(qq, alpha, D, w, lo, full) || !(near == full)) {
      if (++bad < 5)
        std::printf("%s R %g r %g al %g w %g lo %g: near %.9g full %.9g\n", name, double(R), r, al, double(w), double(lo), double(near), double(full));
    }
  }
  std::printf("%s taken %ld outward %ld inward %ld different %ld\n", name, taken, outward, inward, bad);
  return bad || outward < total / 20 || inward < total / 100;
}

int main() { return check<float>("float") | check<double>("double"); }
