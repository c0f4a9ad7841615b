// Host build of the number of states' grid index and volume form (tetra_nos_device.h). Test harness only: compiled by
// tests/test_spline_edges_host.py with g++ and linked with the oracle library.
//
// energy_index against the comparison of e with every e0 + (j + joff) de in long double, over FP32 energies on, next to
// and off grid energies: "index <cases> <wrong>". corner_nos on random tetrahedra, some with equal corners, against the
// oracle's number of states between their ends: "volumes <max error relative to the tetrahedron's volume>".
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <random>

#include "tetra_nos_device.h"

extern "C" double tetra_oracle_tet_nos(const double e[4], const double b[4], double E, double vol);

using namespace tetra;

int main() {
  std::mt19937 rng(11);
  long cases = 0, wrong = 0;
  const int ne = 64;
  for (int it = 0; it < 20000; ++it) {
    const float de = it % 2 ? (float)(1 + rng() % 400) / 128.0f : (float)(rng() % 1000000 + 1) * 3.1e-6f;
    const float e0 = it % 3 ? 0.0f : (float)((int)(rng() % 64) - 32) * 0.25f;
    const double joff = it % 5 == 4 ? -0.5 : 0.0;
    float e = (float)(e0 + ((int)(rng() % 72) - 4 + joff) * (double)de);
    if (it % 4 == 1) e = std::nextafter(e, 1e30f);
    if (it % 4 == 2) e = std::nextafter(e, -1e30f);
    if (it % 4 == 3) e += de * 0.3f;
    for (bool above : {false, true}) {
      int want = ne;
      for (int j = 0; j < ne; ++j) {
        const long double E = (long double)e0 + ((long double)j + joff) * (long double)de;
        if (above ? E > e : E >= e) {
          want = j;
          break;
        }
      }
      int got = (int)energy_index(e, e0, de, 1.0 / (double)de, joff, above, 0.0, (double)ne);
      if (above && want == 1 && got == 0) got = 1;  // a first energy exactly on the grid's: nothing to add there
      ++cases;
      wrong += got != want;
    }
  }
  std::printf("index %ld %ld\n", cases, wrong);
  std::uniform_real_distribution<double> U(0.0, 1.0);
  double worst = 0.0;
  for (int it = 0; it < 20000; ++it) {
    float f[4];
    for (auto& v : f) v = (float)U(rng);
    if (it % 4 == 1) f[1] = f[0];
    if (it % 8 == 2) f[3] = f[2] = f[1];
    std::sort(f, f + 4);
    if (!(f[3] > f[0])) continue;
    const double e[4] = {f[0], f[1], f[2], f[3]}, b[4] = {U(rng), U(rng), U(rng), U(rng)};
    const double E = e[0] + (e[3] - e[0]) * U(rng);
    double w[4], sum = 0.0;
    corner_nos(nos_volumes(f), 1.0, E, w);
    for (int l = 0; l < 4; ++l) sum += b[l] * w[l];
    worst = std::max(worst, std::fabs(sum - tetra_oracle_tet_nos(e, b, E, 4.0)));
  }
  std::printf("volumes %.3e\n", worst);
  return 0;
}
