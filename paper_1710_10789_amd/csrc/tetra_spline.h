// Spline form of the tetrahedron sums (gfx950). Internal header; also built for the host by the tests.
//
// As a function of the energy a tetrahedron's contribution sum_l b_l dw_l/dE (Sec. II.C of Guterding &
// Jeschke, arXiv:1710.10789) is a cubic spline with its four corner energies as knots (a corner weight
// is the density of a barycentric coordinate, i.e. a B-spline with that corner's knot doubled). In the
// basis of truncated powers (Curry and Schoenberg 1966) every corner p contributes one term,
//     12 V P_p b_p (E - E_p)_+^2 + 4 V P_p sum_q (b_q - b_p) / (E_q - E_p) (E - E_p)_+^3,
//     P_p = prod_q 1 / (E_q - E_p)  (q: the three other corners, differences signed, V = V_T/(4 V_G)),
// whatever the order of the corner energies: no sort and no energy cases. The terms of the 24
// tetrahedra around a grid point share the point's knot, so a grid point of a band needs one quadratic
// and one cubic coefficient per orbital for all of them together:
//     T = sum_t 3 P_t,   M_u = sum_{t containing u} P_t r_u   (r_u = 1 / (E_u - E_p), u: 14 neighbours)
//     DOS_m(E) = sum_p 4 V [ T b_p (E - E_p)_+^2 + sum_u M_u (b_u - b_p) (E - E_p)_+^3 ].
// On the equidistant grid the fourth differences of a truncated power vanish but for four entries next
// to its knot, so a point adds four entries per orbital to a histogram and four running sums over the
// histogram give the DOS: no loop over the energies of a window.
//
// The terms of one tetrahedron cancel above its highest knot, which costs digits: relative to the
// tetrahedron's own density about 2^-53 J^3 / (m^2 s) with J the number of energies of the sums, m its
// smallest gap between corner energies and s its smaller second difference (E31 or E42), all in grid
// steps. So all of it runs in FP64 (as fast as FP32 without packed instructions on this chip), and
// tetrahedra with nearly equal corner energies (kDegenerate) are left out here and summed energy
// by energy with the forms of tetra_device.h.
//
// Energies here are in grid steps, u = (E - e0) / de. A point outside the tile is staged at kFarKnot:
// its r_u, about 1e-30, removes the tetrahedra that contain it.
#pragma once

#include "tetra_device.h"

namespace tetra {

constexpr int kNeighbours = 14;
constexpr double kFarKnot = 1.0e30;

// Offsets (axis 1, 2, 3) of the grid points that share a tetrahedron of Table I with a point: the seven
// edge directions of the cube's six tetrahedra, then their negatives.
__host__ __device__ __forceinline__ void neighbour_offset(int u, int& dx, int& dy, int& dz) {
  constexpr signed char D[7][3] = {{1, 0, 0}, {0, 1, 0}, {0, 0, 1}, {1, -1, 0}, {1, 0, 1}, {0, -1, 1}, {1, -1, 1}};
  const int s = u < 7 ? 1 : -1, d = u < 7 ? u : u - 7;
  dx = s * D[d][0];
  dy = s * D[d][1];
  dz = s * D[d][2];
}

// 1/x to FP64 accuracy: the hardware estimate and one third-order step on the device.
__host__ __device__ __forceinline__ double rcp64(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
  const double r = __builtin_amdgcn_rcp(x);
  const double e = __builtin_fma(-x, r, 1.0);
  return __builtin_fma(r, __builtin_fma(e, e, e), r);
#else
  return 1.0 / x;
#endif
}

// m^2 s min(width, E41) of a tetrahedron from its corner energies in units of which a grid step has `width`, in two
// sorted pairs (a0 <= a1, b0 <= b1); the kernels' unit is a power of two (step_unit), so that the differences are those
// of the energies as they are: exact for nearly equal ones, which in grid steps or from an origin of their own would be
// rounded at the scale of that. Zero for two equal finite corners, also beside infinite ones. (A tetrahedron narrower
// than a grid step is held to an error relative to its states per step, not to its own density.)
__host__ __device__ __forceinline__ float spline_gap(float a0, float a1, float b0, float b1, float width = 1.0f) {
  const float e1 = fminf(a0, b0), e4 = fmaxf(a1, b1), c = fmaxf(a0, b0), d = fminf(a1, b1);
  const float e2 = fminf(c, d), e3 = fmaxf(c, d);
  const float m = fminf(fminf(e2 - e1, e3 - e2), e4 - e3);
  return m * m * fminf(fminf(e3 - e1, e4 - e2), 3.0e38f) * fminf(e4 - e1, width);
}
// The power of two 2^k with which the grid step de times 2^k lies in [1, 2).
__host__ __device__ __forceinline__ float step_unit(float de) {
  union {
    float f;
    uint32_t u;
  } x;
  x.f = de;
  x.u = (254u << 23) - (x.u & 0x7f800000u);
  return x.f;
}
// A tetrahedron is left to the energy-by-energy sum where its spline_gap is below this times J^3 (width^4): its terms
// would lose more than the share given of its own density at the far end of the sums. Plain sums end in
// FP32 additions and their errors average over the tetrahedra; exact ones hold 51 bits.
// The plain sums of large problems divide theirs by up to ten (forward_args): the share of the density grows to 2e-3,
// that of the tetrahedra falls to 0.005 %, and more of them average.
constexpr float kDegenerate = 2.2e-12f;       // 2e-4 of the density; 0.05 % of the tetrahedra of generic bands
constexpr float kDegenerateExact = 1.0e-10f;  // 4e-6; 0.4 %

// The tetrahedra of a cube that the spline form leaves out, those with a spline_gap below the limit: bit t for
// tetrahedron t of Table I, and the same of those with finite corners only, which are to be summed another way.
// f: the energies of the corners by slot, +infinity for one that is not finite. A tetrahedron with such a corner contributes
// nothing; its far knot sees to that as long as no two of its other corners are equal, so it is left out as well
// where they are (an edge next to the tile's end may belong to no other tetrahedron of the tile).
__host__ __device__ __forceinline__ uint32_t left_out(const float f[8], float limit, uint32_t& finite, float width = 1.0f) {
  // Corners 2 and 5 belong to all six tetrahedra, the other two run around them.
  constexpr int I[6][2] = {{0, 1}, {1, 3}, {0, 4}, {3, 7}, {4, 6}, {6, 7}};
  const float d0 = fminf(f[2], f[5]), d1 = fmaxf(f[2], f[5]);
  float g[6];
#pragma unroll
  for (int t = 0; t < 6; ++t) {
    const float a = f[I[t][0]], b = f[I[t][1]];
    g[t] = spline_gap(d0, d1, fminf(a, b), fmaxf(a, b), width);
  }
  uint32_t out = 0u;
  finite = 0u;
  if (fminf(fminf(fminf(g[0], g[1]), fminf(g[2], g[3])), fminf(g[4], g[5])) >= limit) return out;
#pragma unroll
  for (int t = 0; t < 6; ++t) {
    if (g[t] >= limit) continue;
    out |= 1u << t;
    if (fmaxf(d1, fmaxf(f[I[t][0]], f[I[t][1]])) < __builtin_huge_valf()) finite |= 1u << t;
  }
  return out;
}

// Nothing is scheduled across it on the device (to bound the registers of long straight-line code).
__host__ __device__ __forceinline__ void schedule_fence() {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_sched_barrier(0);
#endif
}

// M_u (r_u in and M_u out) and T of a point from its 14 reciprocals, all tetrahedra taken part. The
// tetrahedra that contain neighbour u correspond to the edges of its ring (the neighbours that form a
// triangle with u, in cyclic order), M_u = r_u^2 sum over ring edges r_v r_w; the sums over a ring of
// four or six factor.
__host__ __device__ __forceinline__ double knot_coefs(double r[kNeighbours]) {
  auto ring4 = [&](int a, int b, int c, int d) { return (r[a] + r[c]) * (r[b] + r[d]); };
  auto ring6 = [&](int a, int b, int c, int d, int e, int f) {
    return __builtin_fma(r[f], r[e] + r[a], __builtin_fma(r[d], r[c] + r[e], r[b] * (r[a] + r[c])));
  };
  double t[kNeighbours] = {ring6(1, 4, 6, 3, 9, 12),  ring6(0, 4, 2, 10, 13, 12), ring6(7, 10, 1, 4, 6, 5),
                           ring4(8, 6, 0, 9),         ring4(0, 1, 2, 6),          ring4(8, 7, 2, 6),
                           ring6(8, 3, 0, 4, 2, 5),   ring6(10, 2, 5, 8, 11, 13), ring6(3, 6, 5, 7, 11, 9),
                           ring6(11, 13, 12, 0, 3, 8), ring4(7, 2, 1, 13),        ring4(9, 13, 7, 8),
                           ring4(9, 13, 1, 0),        ring6(11, 9, 12, 1, 10, 7)};
  double T = 0.0;
#pragma unroll
  for (int u = 0; u < kNeighbours; ++u) {
    t[u] *= r[u];  // sum of P over the tetrahedra that contain u
    T += t[u];
  }
#pragma unroll
  for (int u = 0; u < kNeighbours; ++u) r[u] *= t[u];
  return T;
}

// The same with the tetrahedra of `skip` left out: bit 4 t + l says that tetrahedron t of the cube in
// which the point is t's l-th corner does not take part. Equal energies (no finite reciprocal) occur
// only in those.
__host__ __device__ __forceinline__ double knot_coefs_skip(double r[kNeighbours], uint32_t skip) {
  constexpr signed char I[24][3] = {
      {0, 1, 4},   {7, 10, 2}, {8, 3, 6},  {11, 9, 13}, {10, 1, 2},  {3, 0, 6},   {8, 7, 5},  {9, 13, 12},
      {1, 2, 4},   {8, 5, 6},  {9, 12, 0}, {11, 13, 7}, {0, 6, 4},   {7, 5, 2},   {13, 12, 1}, {11, 9, 8},
      {5, 6, 2},   {12, 0, 1}, {13, 7, 10}, {9, 8, 3},  {6, 2, 4},   {13, 10, 1}, {9, 3, 0},  {11, 8, 7}};
  double t[kNeighbours], T = 0.0;
#pragma unroll
  for (int u = 0; u < kNeighbours; ++u) {
    t[u] = 0.0;
    r[u] = fabs(r[u]) < 1.0e200 ? r[u] : 0.0;
  }
#pragma unroll
  for (int i = 0; i < 24; ++i) {
    const double p = r[I[i][0]] * r[I[i][1]] * r[I[i][2]];
    const double P = ((skip >> i) & 1u) ? 0.0 : p;
    T += P;
#pragma unroll
    for (int k = 0; k < 3; ++k) t[I[i][k]] += P;
    schedule_fence();  // one at a time: fewer registers
  }
#pragma unroll
  for (int u = 0; u < kNeighbours; ++u) r[u] *= t[u];
  return 3.0 * T;
}

// Fourth differences of the truncated powers x_+^3 and x_+^2 on the grid x, x + 1, x + 2, ... (x: the
// distance of the first grid energy at or above the knot from it): N[i] and n[i] at that energy and the
// three after it, zero from there on.
__host__ __device__ __forceinline__ void knot_differences(double x, double N[4], double n[4]) {
  const double x2 = x * x, x3 = x2 * x, y = 1.0 - x, y2 = y * y;
  N[0] = x3;
  N[1] = __builtin_fma(-3.0, x3, __builtin_fma(3.0, x2, __builtin_fma(3.0, x, 1.0)));
  N[2] = __builtin_fma(3.0, x3, __builtin_fma(-6.0, x2, 4.0));
  N[3] = y2 * y;
  n[0] = x2;
  n[1] = __builtin_fma(-3.0, x2, __builtin_fma(2.0, x, 1.0));
  n[2] = __builtin_fma(3.0, x2, -4.0 * x);
  n[3] = -y2;
}

// The same for the integrated weights (number of states): a tetrahedron's number of states is the quartic
//     V sum_p [ (4/3) T b_p (E - E_p)_+^3 + sum_u M_u (b_u - b_p) (E - E_p)_+^4 ],
// and N[i], n[i] the fifth differences of x_+^4 and x_+^3.
__host__ __device__ __forceinline__ void knot_differences(double x, double N[5], double n[5], bool) {
  double N3[4], n2[4];
  knot_differences(x, N3, n2);
  const double y = 1.0 - x, x2 = x * x, y2 = y * y, p = x2 * x2, q = y2 * y2;
  const double xp = 1.0 + x, yp = 1.0 + y, xp2 = xp * xp, yp2 = yp * yp;
  N[0] = p;
  N[1] = __builtin_fma(-5.0, p, xp2 * xp2);
  N[3] = __builtin_fma(-5.0, q, yp2 * yp2);
  N[4] = q;
  N[2] = 24.0 - ((N[0] + N[1]) + (N[3] + N[4]));
  n[0] = N3[0];
  n[1] = N3[1] - N3[0];
  n[2] = N3[2] - N3[1];
  n[3] = N3[3] - N3[2];
  n[4] = -N3[3];
}

}  // namespace tetra
