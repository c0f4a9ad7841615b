// Host build of the spline form's rule for what it leaves out (left_out, tetra_spline.h). Test harness only:
// compiled by tests/test_spline_edges_host.py with g++ and linked with the oracle library.
//
// A block of 3 x 3 x 3 cubes with energies that no two points share, but for one pair of neighbours with the same
// energy, and one or two points without a finite energy, every placement of the three in the block: the coefficients of
// every finite point are finite, and the sums of the points' entries and of the tetrahedra that were handed on
// agree with the oracle's sum over the tetrahedra with finite corners.
// Prints "ties <placements> <not finite> <max error>", the error relative to the largest sum.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <limits>
#include <random>
#include <vector>

#include "tetra_spline.h"

extern "C" double tetra_oracle_tet_dos(const double e[4], const double b[4], double E, double vol);

using namespace tetra;

int main() {
  constexpr int S = 3, P = S + 1, J = 46, N = P * P * P;
  std::mt19937 rng(7);
  auto at = [](int x, int y, int z) { return (x * P + y) * P + z; };
  std::vector<float> base(N);
  for (int i = 0; i < N; ++i) base[i] = 0.3f + 0.7f * (float)i;
  std::shuffle(base.begin(), base.end(), rng);
  std::vector<double> b(N);
  for (auto& v : b) v = std::uniform_real_distribution<double>(0.1, 1.0)(rng);
  const float inf = std::numeric_limits<float>::infinity();
  long placements = 0, bad = 0;
  double worst = 0.0;
  for (int i = 0; i < N; ++i)
    for (int n = 0; n < 7; ++n) {
      int dx, dy, dz;
      neighbour_offset(n, dx, dy, dz);
      const int X = i / (P * P) + dx, Y = i / P % P + dy, Z = i % P + dz;
      if (X < 0 || X >= P || Y < 0 || Y >= P || Z < 0 || Z >= P) continue;
      const int j2 = at(X, Y, Z);
      for (int k = 0; k < N; ++k) {
        if (k == i || k == j2) continue;
        const int k2 = placements % 3 == 0 ? (int)(rng() % N) : k;  // two bad points now and then
        if (k2 == i || k2 == j2) continue;
        ++placements;
        std::vector<float> u = base;
        u[j2] = u[i];
        u[k] = u[k2] = inf;
        std::vector<uint32_t> skip(N, 0u);
        std::vector<double> want(J, 0.0), got(J, 0.0);
        for (int c = 0; c < S * S * S; ++c) {
          const int x = c / (S * S), y = c / S % S, z = c % S;
          float f[8];
          for (int s = 0; s < 8; ++s) f[s] = u[at(x + (s & 1), y + ((s >> 1) & 1), z + (s >> 2))];
          uint32_t finite;
          const uint32_t out = left_out(f, kDegenerate * J * J * J, finite);
          if (finite & ~out) ++bad;
          for (int t = 0; t < 6; ++t) {
            double e[4], w[4];
            bool fin = true;
            for (int l = 0; l < 4; ++l) {
              const int s = (tet_slots(t) >> (4 * l)) & 7, p = at(x + (s & 1), y + ((s >> 1) & 1), z + (s >> 2));
              e[l] = u[p];
              w[l] = b[p];
              fin = fin && std::isfinite(u[p]);
              if ((out >> t) & 1u) skip[p] |= 1u << (4 * t + l);
            }
            if (((finite >> t) & 1u) && !fin) ++bad;
            if (fin)
              for (int j = 0; j < J; ++j) {
                const double v = tetra_oracle_tet_dos(e, w, (double)j, 4.0);
                want[j] += v;
                if ((finite >> t) & 1u) got[j] += v;
              }
          }
        }
        std::vector<double> h(J + 4, 0.0);
        for (int p = 0; p < N; ++p) {
          if (!std::isfinite(u[p])) continue;
          double r[kNeighbours], bn[kNeighbours];
          for (int m = 0; m < kNeighbours; ++m) {
            neighbour_offset(m, dx, dy, dz);
            const int x = p / (P * P) + dx, y = p / P % P + dy, z = p % P + dz;
            const bool in = x >= 0 && x < P && y >= 0 && y < P && z >= 0 && z < P;
            r[m] = rcp64((in && std::isfinite(u[at(x, y, z)]) ? (double)u[at(x, y, z)] : kFarKnot) - (double)u[p]);
            bn[m] = in ? b[at(x, y, z)] : 0.0;
          }
          const double T = skip[p] ? knot_coefs_skip(r, skip[p]) : knot_coefs(r);
          double Q = 0.0, N4[4], n4[4];
          for (int m = 0; m < kNeighbours; ++m) Q += r[m] * (bn[m] - b[p]);
          if (!std::isfinite(T) || !std::isfinite(Q)) ++bad;
          const double ju = std::ceil((double)u[p]);
          knot_differences(ju - u[p], N4, n4);
          for (int m = 0; m < 4; ++m)
            if ((int)ju + m < J) h[(int)ju + m] += 4.0 * (Q * N4[m] + T * b[p] * n4[m]);
        }
        for (int m = 0; m < 4; ++m)
          for (int j = 1; j < J; ++j) h[j] += h[j - 1];
        double top = 0.0, err = 0.0;
        for (int j = 0; j < J; ++j) {
          top = std::max(top, std::fabs(want[j]));
          err = std::max(err, std::fabs(want[j] - got[j] - h[j]));
        }
        if (!(err <= 1e300)) err = 1e300;
        worst = std::max(worst, err / top);
      }
    }
  std::printf("ties %ld %ld %.3e\n", placements, bad, worst);
  return 0;
}
