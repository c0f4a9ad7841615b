// Host build of the spline form (tetra_spline.h) against the FP64 oracle's tetrahedra. Test harness only:
// compiled by tests/test_spline_host.py with g++ and linked with the oracle library.
//
// Blocks of 3 x 3 x 3 cubes with random energies (in grid steps) and weights, some with equal energies:
// every point's coefficients from its neighbours (points outside the block far away), its entries added
// to a histogram, four running sums, against the sum over the block's tetrahedra of the oracle's
// sum_l b_l dw_l/dE, and the same for the number of states (fifth differences, five sums). Tetrahedra whose spline_gap is below the limit are left out on both sides.
// Prints "block <blocks> <left out> <max error>" and "states <max error>" with the error relative to the largest sum, and the number
// of wrong quotients of the kernels' divisions by constants.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>

#include "tetra_forward_args.h"
#include "tetra_spline.h"

extern "C" double tetra_oracle_tet_nos(const double e[4], const double b[4], double E, double vol);
extern "C" double tetra_oracle_tet_dos(const double e[4], const double b[4], double E, double vol);

using namespace tetra;

int main() {
  constexpr int S = 3, P = S + 1;
  std::mt19937 rng(5);
  std::uniform_real_distribution<double> U(0.0, 40.0), W(-0.2, 1.0);
  double worst = 0.0, worst5 = 0.0;
  long left = 0;
  const int blocks = 60, J = 46;
  auto at = [](int x, int y, int z) { return (x * P + y) * P + z; };
  for (int it = 0; it < blocks; ++it) {
    std::vector<float> u(P * P * P);
    std::vector<double> b(P * P * P);
    for (auto& v : u) v = (float)U(rng);
    for (auto& v : b) v = W(rng);
    if (it % 3 == 1)
      for (int i = 0; i < 6; ++i) u[rng() % u.size()] = u[rng() % u.size()];  // equal energies
    if (it % 3 == 2)
      for (size_t i = 0; i + 4 < u.size(); i += 4) u[i] = u[i + 1] + 1.0e-6f * (float)(rng() % 3);
    std::vector<uint32_t> skip(u.size(), 0u);
    std::vector<double> want(J, 0.0), states(J, 0.0);
    for (int x = 0; x < S; ++x)
      for (int y = 0; y < S; ++y)
        for (int z = 0; z < S; ++z)
          for (int t = 0; t < 6; ++t) {
            const uint32_t slots = tet_slots(t);
            int p[4];
            float f[4];
            double e[4], w[4];
            for (int l = 0; l < 4; ++l) {
              const int s = (slots >> (4 * l)) & 7;
              p[l] = at(x + (s & 1), y + ((s >> 1) & 1), z + (s >> 2));
              e[l] = f[l] = u[p[l]];
              w[l] = b[p[l]];
            }
            const float gap = spline_gap(std::min(f[0], f[1]), std::max(f[0], f[1]), std::min(f[2], f[3]), std::max(f[2], f[3]));
            if (gap < kDegenerate * J * J * J) {
              ++left;
              for (int l = 0; l < 4; ++l) skip[p[l]] |= 1u << (4 * t + l);
              continue;
            }
            for (int j = 0; j < J; ++j) {
              want[j] += tetra_oracle_tet_dos(e, w, (double)j, 4.0);
              states[j] += tetra_oracle_tet_nos(e, w, (double)j, 4.0);
            }
          }
    std::vector<double> h(J + 4, 0.0), h5(J + 5, 0.0);
    for (int x = 0; x < P; ++x)
      for (int y = 0; y < P; ++y)
        for (int z = 0; z < P; ++z) {
          const int p = at(x, y, z);
          double r[kNeighbours], bn[kNeighbours];
          for (int n = 0; n < kNeighbours; ++n) {
            int dx, dy, dz;
            neighbour_offset(n, dx, dy, dz);
            const int X = x + dx, Y = y + dy, Z = z + dz;
            const bool in = X >= 0 && X < P && Y >= 0 && Y < P && Z >= 0 && Z < P;
            r[n] = rcp64((in ? (double)u[at(X, Y, Z)] : kFarKnot) - (double)u[p]);
            bn[n] = in ? b[at(X, Y, Z)] : 0.0;
          }
          const double T = skip[p] ? knot_coefs_skip(r, skip[p]) : knot_coefs(r);
          double Q = 0.0, N[4], n4[4];
          for (int n = 0; n < kNeighbours; ++n) Q += r[n] * (bn[n] - b[p]);
          const double ju = std::ceil((double)u[p]);
          knot_differences(ju - u[p], N, n4);
          for (int i = 0; i < 4; ++i)
            if ((int)ju + i < J) h[(int)ju + i] += 4.0 * (Q * N[i] + T * b[p] * n4[i]);
          double N5[5], n5[5];
          knot_differences(ju - u[p], N5, n5, true);
          for (int i = 0; i < 5; ++i)
            if ((int)ju + i < J) h5[(int)ju + i] += Q * N5[i] + 4.0 / 3.0 * T * b[p] * n5[i];
        }
    for (int k = 0; k < 4; ++k)
      for (int j = 1; j < J; ++j) h[j] += h[j - 1];
    for (int k = 0; k < 5; ++k)
      for (int j = 1; j < J; ++j) h5[j] += h5[j - 1];
    double top = 0.0, err = 0.0;
    for (int j = 0; j < J; ++j) {
      top = std::max(top, std::fabs(want[j]));
      err = std::max(err, std::fabs(want[j] - h[j]));
    }
    worst = std::max(worst, err / top);
    top = err = 0.0;
    for (int j = 0; j < J; ++j) {
      top = std::max(top, std::fabs(states[j]));
      err = std::max(err, std::fabs(states[j] - h5[j]));
    }
    worst5 = std::max(worst5, err / top);
  }
  std::printf("block %d %ld %.3e\n", blocks, left, worst);
  std::printf("states %.3e\n", worst5);
  long bad = 0;
  for (int d : {1, 2, 3, 5, 7, 8, 9, 12, 63, 64, 65, 1000, 1728, 4095, 65537, 1000003, 2147483647}) {
    const FastDiv f = fast_div(d);
    for (long k = 0; k < 4000; ++k) {
      const uint32_t n = (uint32_t)((k < 2000 ? k * 1073741 : 2147483647 - (k - 2000) * 77) & 0x7fffffff);
      for (uint32_t v : {n, (uint32_t)((n / d) * (uint32_t)d)})
        if ((uint32_t)(((uint64_t)v * f.m) >> f.s) != v / (uint32_t)d) ++bad;
    }
  }
  std::printf("division %ld\n", bad);
  return 0;
}
