// Host checks of the reverse sweep at a crossing that the forward fit and the
// sweep may judge differently.
//   step  step_vjp() of a step whose surface is out of reach passes zeros back.
#include <cmath>
#include <cstdio>
#include <cstring>

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

}  // namespace

int main(int argc, char** argv) {
  if (argc == 2 && !std::strcmp(argv[1], "step")) return unreachable_step<float>() | unreachable_step<double>();
  return 2;
}
