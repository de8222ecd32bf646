// The FP64 surface-frame update on given states and hits, in a host build.
// Reads records of 33 float64 from argv[1] (kind, tx, ty, state 6, packed 5x5
// covariance 15, hit 3, packed hit covariance 6) and writes records of 23 to
// argv[2] (taken by update5, state 6, covariance 15, chi2).
#include <cstdint>
#include <cstdio>

#include "kf_surface.hpp"

int main(int argc, char** argv) {
  if (argc != 3) return 2;
  FILE* in = std::fopen(argv[1], "rb");
  FILE* out = std::fopen(argv[2], "wb");
  if (!in || !out) return 2;
  double r[33], w[23];
  while (std::fread(r, sizeof(double), 33, in) == 33) {
    kf::SurfState<double> s;
    s.kind = int(r[0]);
    s.tx = r[1];
    s.ty = r[2];
    s.q = 1;
    for (int i = 0; i < 6; ++i) s.p[i] = r[3 + i];
    for (int i = 0; i < 15; ++i) s.c[i] = r[9 + i];
    uint32_t st = 0;
    w[22] = 0.0;
    w[0] = kf::update5(s, r + 24, r + 27, w[22], st) ? 1.0 : 0.0;
    for (int i = 0; i < 6; ++i) w[1 + i] = s.p[i];
    for (int i = 0; i < 15; ++i) w[7 + i] = s.c[i];
    if (std::fwrite(w, sizeof(double), 23, out) != 23) return 2;
  }
  std::fclose(in);
  return std::fclose(out) ? 2 : 0;
}
