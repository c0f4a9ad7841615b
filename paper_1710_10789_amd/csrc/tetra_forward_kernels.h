// Forward kernels: orbital-resolved tetrahedron DOS on gfx950.
//
// Sum of eq. (tetracontriborbitalresolved) over the tetrahedra and bands of a periodic k-grid
// (eq. tetmethoorbitalresolved, Guterding & Jeschke, arXiv:1710.10789, Sec. II.C), with the
// tetrahedra of Table I.
//
// Work decomposition: one workgroup per (tile of at most 8 x 8 x 8 cubes, band). The tile's grid points
// (9 x 9 x 9: 1.42 points per cube; 4 x 4 x 16 cubes have 1.66) are staged once in LDS, energies and
// orbital weights. Then, into one LDS histogram (FP64 atomics, 8 lane-adds per clock and CU against 0.3 for FP32 ones):
//  * the spline form (tetra_spline.h): one lane per grid point forms the coefficients of the point's truncated powers
//    from all tetrahedra of the tile around it and adds four entries per orbital, fourth differences; four running
//    sums down the histogram give the tile's DOS. The work per tile does not depend on the energy windows:
//    64^3 x 8 x 8 x 1000 took 0.32 ms with a loop over every tetrahedron's window and takes 0.171 ms;
//    24^3 x 8 x 8 x 4096, with windows of 75 energies, 0.04 ms. Bound by FP64 issue (about 560 instructions per point,
//    516 of them FP64), the LDS (120 weight reads and 32 atomics per point of 8 orbitals) and the latencies of a
//    unit's stages, of which two units per CU hide only part: each microsecond of the about 20 of a unit counts.
//  * tetrahedra with nearly equal corner energies, energy by energy onto those sums (sum_tets): a few of generic bands,
//    through a queue; hundreds to all of them where a lattice's symmetry or a band without dispersion along an axis
//    makes energies equal. Four bands of 8 orbitals, 1000 energies, loop over every tetrahedron's window -> the form
//    that threw the tile's spline form away for such a loop -> this: nearest neighbours on a simple cubic lattice 64^3
//    0.28, 0.24, 0.18 ms, fcc 0.52, 0.34, 0.21 ms, layered 0.78, 0.92, 0.75 ms.
//    So is everything in a tile-band whose energy range the histogram does not hold (thousands of energies) or with
//    weights that are not finite.
// One global float atomic per touched (energy, orbital) bin when the workgroup finishes.
// Workgroups are assigned so that each XCD (eight per MI355X, each with its own L2) works through a
// contiguous range of tiles of the same band, keeping shared halo points in one L2.
// No kernel here may spill vector registers: the compiler has placed such stores behind a loop's exit
// with no lane active.

#pragma once

#include <type_traits>

#include "tetra_device.h"
#include "tetra_forward_args.h"
#include "tetra_nos_device.h"
#include "tetra_spline_tile.h"
#include "tetra_weights.h"
#include "tetra_window_kernels.h"

namespace tetra {

namespace {

// The bound of the exact mode for one work unit; every lane of the workgroup calls it: the exponent of
// B = sum 12 V bmax / E41 over the tetrahedra with a possibly non-empty window into *gexp (atomicMax: independent of the
// order). A tetrahedron's DOS never exceeds 3 V_T / (V_G E41), so no bin's |sum| over the unit exceeds B.
template <int NORB>
struct BoundShared {
  float eps[NP];
  float red[3 * NWMAX];
};
template <int NORB, typename WT>
__device__ __forceinline__ void bound_unit(const FwdArgs& a, int unit, BoundShared<NORB>& sh) {
  int band;
  const Tile tl = unit_tile(a, unit, band);
  const int qy = tl.cy + 1, qz = tl.cz + 1, np = (tl.cx + 1) * qy * qz, ncubes = tl.cx * tl.cy * tl.cz;
  const int by_qz = small_inverse(qz), by_qy = small_inverse(qy);
  const int tid = threadIdx.x, NT = blockDim.x, NW = NT >> 6;
  const int64_t nk = (int64_t)a.n1 * a.n2 * a.n3;
  const float* eps_n = a.eps + (int64_t)band * nk;
  const WT* w_n = static_cast<const WT*>(a.w) + (int64_t)band * NORB * nk;
  const float wscale = a.w_scale ? a.w_scale[band] : 1.0f;
  float lmin = __builtin_huge_valf(), lmax = -__builtin_huge_valf(), lbmax = 0.0f;
  for (int q = tid; q < np; q += NT) {
    const int r = small_div(q, by_qz), pz = q - r * qz, px = small_div(r, by_qy), py = r - px * qy;
    const int64_t k = ((int64_t)wrap(tl.x0 + px, a.n1) * a.n2 + wrap(tl.y0 + py, a.n2)) * a.n3 + wrap(tl.z0 + pz, a.n3);
    const float e = eps_n[k];
    sh.eps[px * PY + py * PZ + pz] = e;
    if (__builtin_isfinite(e)) {
      lmin = fminf(lmin, e);
      lmax = fmaxf(lmax, e);
    }
#pragma unroll
    for (int m = 0; m < NORB; ++m) lbmax = fmaxf(lbmax, fabsf(weight_value(w_n[(int64_t)m * nk + k], wscale)));
  }
  lmin = wave_min(lmin);
  lmax = wave_max(lmax);
  lbmax = wave_max(lbmax);
  if ((tid & 63) == 0) {
    sh.red[tid >> 6] = lmin;
    sh.red[NW + (tid >> 6)] = lmax;
    sh.red[2 * NW + (tid >> 6)] = lbmax;
  }
  __syncthreads();
  float emin = sh.red[0], emax = sh.red[NW], bmax = sh.red[2 * NW];
  for (int i = 1; i < NW; ++i) {
    emin = fminf(emin, sh.red[i]);
    emax = fmaxf(emax, sh.red[NW + i]);
    bmax = fmaxf(bmax, sh.red[2 * NW + i]);
  }
  if (!(emin <= emax)) return;  // no finite energy
  int J0, J1;
  range_window(emin, emax, a.e0, a.inv_de, a.ne, J0, J1);
  float bound = 0.0f;
  const float c12 = 12.0f * a.V * bmax;
  for_lanes(ncubes, [&](int c) {
    const int r = c / tl.cz, iz = c - r * tl.cz, ix = r / tl.cy, iy = r - ix * tl.cy;
    const float* fc = &sh.eps[ix * PY + iy * PZ + iz];
#pragma unroll 1
    for (int t = 0; t < 6; ++t) {
      const uint32_t slots = tet_slots(t);
      float lo = __builtin_huge_valf(), hi = -__builtin_huge_valf();
      bool fin = true;
#pragma unroll
      for (int l = 0; l < 4; ++l) {
        const int s = (slots >> (4 * l)) & 7;
        const float e = fc[(s & 1) * PY + ((s >> 1) & 1) * PZ + (s >> 2)];
        fin = fin && __builtin_isfinite(e);
        lo = fminf(lo, e);
        hi = fmaxf(hi, e);
      }
      if (!fin || !(hi > lo)) continue;
      int jlo, jhi;
      energy_window(lo, hi, a.e0, a.inv_de, J0, J1, jlo, jhi);
      if (jlo <= jhi + 2) bound += c12 * rcp(hi - lo);
    }
  });
  bound = wave_sum(fminf(bound, 1.0e37f));
  __syncthreads();  // every lane has read sh.red
  if ((tid & 63) == 0) sh.red[tid >> 6] = bound;
  __syncthreads();
  float B = 0.0f;
  for (int i = 0; i < NW; ++i) B += sh.red[i];
  if (!(B > 0.0f) || tid != 0) return;
  int be;
  frexpf(fminf(B, 3.0e38f), &be);
  atomicMax(a.gexp, be);
}

// ---------------------------------------------------------------------------------------------
// Spline form (tetra_spline.h): one lane per grid point of the tile instead of one per cube.

template <int NORB>
struct SplineFixed {
  double u[kKnotPad];  // knots: energies in grid steps
  float f[NP];         // the energies times `unit`, for the search for degenerate tetrahedra; infinite where not finite
  float wlo[kWeightPad];
  float w[NP * NORB];
  float whi[kWeightPad];
  uint32_t skip[NP];
  unsigned short queue[kQueue];
  float red[3 * NWMAX];
  double dred[NWMAX];
  int nq, nout;  // left-out tetrahedra with finite corners, all of them
};
template <int NORB>
constexpr int spline_words() { return (kLdsBytes - 64 - (int)sizeof(SplineFixed<NORB>)) / 8; }
template <int NORB>
struct SplineShared : SplineFixed<NORB> {
  double hist[spline_words<NORB>()];
};

// One work unit; every lane of the workgroup calls it.
// MODE 0: FP64 sums, flushed with float atomics. MODE 2: 64-bit integers, so that nothing depends on the
// order of the atomics: a first sweep over the points finds the largest entry, which fixes the scale.
// MODE 3: the increments N(E_j) - N(E_{j-1}) of the number of states on the grid e0 + (j + joff) de
// (everything below the grid at index 0) instead of the DOS: fifth differences of quartics, and the same
// four running sums.
template <int NORB, typename WT, int MODE>
__device__ __forceinline__ void spline_unit(const FwdArgs& a, int unit, SplineShared<NORB>& sh) {
  using Acc = typename std::conditional<MODE == 2, long long, double>::type;
  constexpr bool INC = MODE == 3;
  constexpr int NE = INC ? 5 : 4;  // entries of a point
  int band;
  const Tile tl = unit_tile(a, unit, band);
  const int x0 = tl.x0, y0 = tl.y0, z0 = tl.z0, cy = tl.cy, cz = tl.cz;
  const int qy = cy + 1, qz = cz + 1, np = (tl.cx + 1) * qy * qz, ncubes = tl.cx * cy * cz;
  const int by_qz = small_inverse(qz), by_qy = small_inverse(qy);
  const int tid = threadIdx.x, NT = blockDim.x, NW = NT >> 6;
  const int64_t nk = (int64_t)a.n1 * a.n2 * a.n3;
  const float* eps_n = a.eps + (int64_t)band * nk;
  const WT* w_n = static_cast<const WT*>(a.w) + (int64_t)band * NORB * nk;
  const float wscale = a.w_scale ? a.w_scale[band] : 1.0f;
  const double e0 = a.e0d, inv_de = a.inv_ded, joff = INC ? a.joff : 0.0;
  auto split = [&](int q, int& px, int& py, int& pz) {
    const int r = small_div(q, by_qz);
    pz = q - r * qz;
    px = small_div(r, by_qy);
    py = r - px * qy;
  };

  // The loads of a lane's first two points are all in flight while the LDS is prepared: 0.174 -> 0.167 ms at
  // 64^3 x 8 x 8 x 1000 (staging and the search below alone: 55 -> 44 us) against one point after the other.
  auto grid_index = [&](int px, int py, int pz) {
    return ((uint32_t)wrap(x0 + px, a.n1) * a.n2 + wrap(y0 + py, a.n2)) * a.n3 + wrap(z0 + pz, a.n3);
  };
  float ahead_e[2];
  WT ahead_w[2][NORB];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int q = tid + i * NT;
    if (q < np) {
      int px, py, pz;
      split(q, px, py, pz);
      const uint32_t k = grid_index(px, py, pz);
      ahead_e[i] = eps_n[k];
#pragma unroll
      for (int m = 0; m < NORB; ++m) ahead_w[i][m] = (w_n + (int64_t)m * nk)[k];
    }
  }
  for_lanes(kKnotPad, [&](int i) { sh.u[i] = kFarKnot; });
  for_lanes(kWeightPad, [&](int i) { sh.wlo[i] = sh.whi[i] = 0.0f; });
  for_lanes(NP, [&](int i) { sh.skip[i] = 0u; });
  if (np < NP)  // every word a neighbour offset can reach holds a finite value
    for_lanes(NP * NORB, [&](int i) { sh.w[i] = 0.0f; });
  if (tid == 0) sh.nq = sh.nout = 0;
  __syncthreads();
  float lmin = __builtin_huge_valf(), lmax = -__builtin_huge_valf(), lbmax = 0.0f, lsum = 0.0f;
  auto stage = [&](int q, float e, auto&& weight) {
    int px, py, pz;
    split(q, px, py, pz);
    const int p = px * PY + py * PZ + pz;
    const bool good = __builtin_isfinite(e);
    sh.f[p] = good ? e * a.unit : __builtin_huge_valf();
    if (good) {
      sh.u[kKnotMargin + px * SY + py * SZ + pz] = ((double)e - e0) * inv_de - joff;
      lmin = fminf(lmin, e);
      lmax = fmaxf(lmax, e);
    }
#pragma unroll
    for (int m = 0; m < NORB; ++m) {
      const float b = weight_value(weight(m), wscale);
      sh.w[m * NP + p] = b;
      lbmax = fmaxf(lbmax, fabsf(b));
      lsum += b;  // not a number when one of them is none
    }
  };
#pragma unroll
  for (int i = 0; i < 2; ++i)
    if (tid + i * NT < np) stage(tid + i * NT, ahead_e[i], [&](int m) { return ahead_w[i][m]; });
  for (int q0 = 2 * NT; q0 < np; q0 += NT) {  // only tiles one cube thick have so many points per lane
    const int q = q0 + tid;
    if (q < np) {
      int px, py, pz;
      split(q, px, py, pz);
      const uint32_t k = grid_index(px, py, pz);
      stage(q, eps_n[k], [&](int m) { return (w_n + (int64_t)m * nk)[k]; });
    }
  }
  if (!(fabsf(lsum) < __builtin_huge_valf())) lbmax = __builtin_huge_valf();
  lmin = wave_min(lmin);
  lmax = wave_max(lmax);
  lbmax = wave_max(lbmax);
  if ((tid & 63) == 0) {
    sh.red[tid >> 6] = lmin;
    sh.red[NW + (tid >> 6)] = lmax;
    sh.red[2 * NW + (tid >> 6)] = lbmax;
  }
  __syncthreads();
  float emin = sh.red[0], emax = sh.red[NW], bmax = sh.red[2 * NW];
  for (int i = 1; i < NW; ++i) {
    emin = fminf(emin, sh.red[i]);
    emax = fmaxf(emax, sh.red[NW + i]);
    bmax = fmaxf(bmax, sh.red[2 * NW + i]);
  }
  emin = uniform(emin);
  emax = uniform(emax);
  if (!(emin <= emax)) return;  // no finite energy
  const double umin = ((double)emin - e0) * inv_de - joff, umax = ((double)emax - e0) * inv_de - joff;
  auto index = [&](float e, bool above, double lo, double top) {  // INC
    return energy_index(e, e0, a.ded, inv_de, joff, above, lo, top);
  };
  // above the energy grid (a flat tetrahedron on its last energy has all its states there)
  if (INC ? index(emin, false, -1.0, a.ned) > (a.ned - 1.0) : !(umin < (a.ned - 1.0))) return;
  if (!(umax > 0.0)) {  // below it
    if (INC && a.shift == 0) {
      // every state counts at index 0: each finite tetrahedron gives V times its corners' weights
      for_lanes(NORB, [&](int m) { sh.hist[m] = 0.0; });
      __syncthreads();
      for (int m = 0; m < NORB; ++m) {
        double sum = 0.0;
        for_lanes(ncubes, [&](int c) {
          const int r = c / cz, iz = c - r * cz, ix = r / cy, iy = r - ix * cy, p = ix * PY + iy * PZ + iz;
#pragma unroll
          for (int t = 0; t < 6; ++t) {
            const uint32_t slots = tet_slots(t);
            float top = -__builtin_huge_valf(), b = 0.0f;
#pragma unroll
            for (int l = 0; l < 4; ++l) {
              const int s = (slots >> (4 * l)) & 7, q = p + (s & 1) * PY + ((s >> 1) & 1) * PZ + (s >> 2);
              top = fmaxf(top, sh.f[q]);
              b += sh.w[m * NP + q];
            }
            sum += top < __builtin_huge_valf() && b == b ? (double)b : 0.0;
          }
        });
        if (sum != 0.0) unsafeAtomicAdd(&sh.hist[m], sum);
      }
      __syncthreads();
      for_lanes(NORB, [&](int m) { atomic_add_global(&a.dos[m], (float)(sh.hist[m] * a.Vd)); });
    }
    return;
  }
  // Rows of the sums: from the first grid energy at or above the lowest knot (below the grid's first
  // energy too) to the last one below the highest (the first at or above it for the increments).
  const double rows_d = INC ? fmin(fmax(ceil(umax), index(emax, false, -1.0, a.ned)), (a.ned - 1.0)) + 1.0 - floor(umin)
                            : fmin(ceil(umax), a.ned) - floor(umin);
  // Energy ranges beyond the histogram and weights that are not finite: every tetrahedron energy by energy.
  const bool finite = uniform(bmax) < 3.0e38f;
  const bool direct = !(rows_d + NE + 2 <= (double)spline_words<NORB>()) || !finite;
  const int base = direct ? 0 : uniform((int)floor(umin)), rows = direct ? 0 : uniform((int)rows_d);
  const float J = (float)rows, limit = (MODE == 2 ? a.degenerate_exact : a.degenerate) * J * J * J;

  // Degenerate tetrahedra: their bits at their corner points, and a queue of those with finite
  // corners, as far as it goes.
  const int by_cz = small_inverse(cz), by_cy = small_inverse(cy);
  if (!direct) for_lanes(ncubes, [&](int c) {
    const int r = small_div(c, by_cz), iz = c - r * cz, ix = small_div(r, by_cy), iy = r - ix * cy;
    const float* fc = &sh.f[ix * PY + iy * PZ + iz];
    float f[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) f[s] = fc[(s & 1) * PY + ((s >> 1) & 1) * PZ + (s >> 2)];
    uint32_t whole;
    const uint32_t out = left_out(f, limit, whole, a.width);
    if (out) {
      atomicAdd(&sh.nout, __popc(out));
      int at = atomicAdd(&sh.nq, __popc(whole));
#pragma unroll
      for (int t = 0; t < 6; ++t) {
        if (!((out >> t) & 1u)) continue;
        if (((whole >> t) & 1u) && at < kQueue) sh.queue[at++] = (unsigned short)(c * 6 + t);
        const uint32_t slots = tet_slots(t);
#pragma unroll
        for (int l = 0; l < 4; ++l) {
          const int s = (slots >> (4 * l)) & 7;
          const int p = (ix + (s & 1)) * PY + (iy + ((s >> 1) & 1)) * PZ + iz + (s >> 2);
          atomicOr(&sh.skip[p], 1u << (4 * t + l));
        }
      }
    }
  });
  __syncthreads();
  const int nq = direct ? 6 * ncubes : uniform(sh.nq);
  const bool none = direct || uniform(sh.nout) == 6 * ncubes;  // nothing in the spline form

  // As many orbitals at a time as the histogram holds, then as many copies of it (a lane adds into copy
  // lane mod copies: neighbouring points often share a bin). Energy by energy alone: all orbitals, some energies at a time.
  int group = NORB, RS = (rows + NE + 1) | 1;
  int J0 = base, J1 = base + rows - 1;
  if (direct) {
    const double top = (a.ned - 1.0);
    J0 = uniform((int)fmax(INC ? index(emin, false, 0.0, top) : floor(umin), 0.0));
    J1 = uniform((int)fmin(INC ? index(emax, false, 0.0, top) : ceil(umax), top));
    RS = (spline_words<NORB>() / NORB - 2) | 1;
  }
  while ((RS * group | 1) > spline_words<NORB>()) group = (group + 1) / 2;
  const int plane = RS * group | 1;  // odd: the copies of a bin in different banks
  const int copies = histogram_copies(plane, spline_words<NORB>());
  Acc* const hist = reinterpret_cast<Acc*>(sh.hist);
  const double c4 = INC ? a.Vd : a.c4;

  // Coefficients of this lane's point q, then act(m, D) with the four entries of every orbital of the
  // group [m0, m1), scaled by `scale`.
  auto point = [&](int q, int m0, int m1, double scale, auto&& act) {
    int px, py, pz;
    split(q, px, py, pz);
    const double* up = &sh.u[kKnotMargin + px * SY + py * SZ + pz];
    const double u0 = up[0];
    const double ju = ceil(u0);
    int b = base;  // opaque, so that no double of it is kept live over the whole unit
    asm volatile("" : "+v"(b));
    const double jr = ju - b;
    if (!(jr < (double)rows)) return;  // above the last row (or not finite)
    double M[kNeighbours];
    const int p = px * PY + py * PZ + pz;
    knot_reciprocals(up, u0, M);
    const uint32_t skip = sh.skip[p];
    const double T = __any(skip != 0u) ? knot_coefs_skip(M, skip) : knot_coefs(M);
    double Ms = 0.0;
#pragma unroll
    for (int u = 0; u < kNeighbours; ++u) Ms += M[u];
    double N[NE], n[NE];
    if constexpr (INC) knot_differences(ju - u0, N, n, true);
    else knot_differences(ju - u0, N, n);
#pragma unroll
    for (int i = 0; i < NE; ++i) {
      N[i] *= scale;
      n[i] *= scale * (INC ? (4.0 / 3.0) * T : T);
    }
    const int row = (int)jr;
    auto orbital = [&](int m) {
      const float* w = sh.w + m * NP + p;
      const double bp = w[0];
      const double Q = knot_contract(M, Ms, w);
      double D[NE];
#pragma unroll
      for (int i = 0; i < NE; ++i) D[i] = __builtin_fma(Q, N[i], bp * n[i]);
      act(m, row, D);
    };
    // two at a time: the next one's weights are on their way (0.167 against 0.174 ms one at a time)
#pragma unroll 2
    for (int m = m0; m < m1; ++m) orbital(m);
  };

  // The `count` tetrahedra of the queue energy by energy, or all that are left out (count: all there are), 2^lg lanes
  // each: the energies [c0, c1] and orbitals [m0, m1) into rows from c0 on, lane i into plane i & planes. MODE 2: times
  // 2^sexp.
  // Next to each other in the tile are tetrahedra with the same energies (all along an axis without dispersion),
  // and FP64 atomics to one address serialise: neighbouring lanes take tetrahedra an eighth of the queue apart, or of
  // cubes of which no two in 64 lie in a line along an axis.
  auto sum_tets = [&](int count, int lg, bool all, int m0, int m1, int c0, int c1, int planes, int sexp) {
    constexpr int G = NORB < 8 ? NORB : 8;  // orbitals whose weights a lane holds
    const double unit = MODE == 2 ? ldexp(1.0, sexp) : 1.0;
    const int eighth = (count + 7) >> 3, area = tl.cx * cy, by_cx = small_inverse(tl.cx);
    const float by_unit = step_unit(a.unit);
    for_lanes((all ? count : 8 * eighth) << lg, [&](int i) {
      const int k = i >> lg, sub = i & ((1 << lg) - 1);
      int t, ix, iy, iz;
      if (all) {
        t = (k >= ncubes) + (k >= 2 * ncubes) + (k >= 3 * ncubes) + (k >= 4 * ncubes) + (k >= 5 * ncubes);
        const int c = k - t * ncubes, z = small_div(small_div(c, by_cx), by_cy), r = c - z * area;
        ix = small_div(r, by_cy);
        iy = r - ix * cy;
        iz = z + ix + iy;
        iz -= small_div(iz, by_cz) * cz;
        const uint32_t skip = sh.skip[ix * PY + (iy + 1) * PZ + iz];  // of corner 2, which all six have
        if (!direct && !((skip >> ((0x14100c090502ull >> (8 * t)) & 31)) & 1u)) return;
      } else {
        const int q = (k & 7) * eighth + (k >> 3);
        if (q >= count) return;
        const int it = sh.queue[q], c = it / 6, r = small_div(c, by_cz);
        t = it - 6 * c;
        iz = c - r * cz;
        ix = small_div(r, by_cy);
        iy = r - ix * cy;
      }
      const uint32_t slots = tet_slots(t);
      float e[4];
      int pt[4];
#pragma unroll
      for (int l = 0; l < 4; ++l) {
        const int s = (slots >> (4 * l)) & 7;
        pt[l] = (ix + (s & 1)) * PY + (iy + ((s >> 1) & 1)) * PZ + iz + (s >> 2);
        e[l] = sh.f[pt[l]] * by_unit;
      }
      if (!finite4(e[0], e[1], e[2], e[3])) return;
      sort4(e, pt);
      if (!INC && !(e[3] > e[0])) return;
      Acc* const h0 = hist + (i & planes) * plane - c0;
#pragma unroll 1
      for (int mc = m0; mc < m1; mc += G) {
        float wt[4][G];
#pragma unroll
        for (int m = 0; m < G; ++m) {
          const int at = min(mc + m, m1 - 1);
#pragma unroll
          for (int l = 0; l < 4; ++l) wt[l][m] = sh.w[at * NP + pt[l]];
          if (!finite) {  // a weight that is no number adds nothing
            const float sum = (wt[0][m] + wt[1][m]) + (wt[2][m] + wt[3][m]);
#pragma unroll
            for (int l = 0; l < 4; ++l) wt[l][m] = sum == sum ? wt[l][m] : 0.0f;
          }
        }
        auto put = [&](int j, const float g[4]) {
          Acc* h = h0 + (mc - m0) * RS + j;
#pragma unroll
          for (int m = 0; m < G; ++m) {
            if (mc + m >= m1) continue;
            const float v = g[0] * wt[0][m] + g[1] * wt[1][m] + g[2] * wt[2][m] + g[3] * wt[3][m];
            if constexpr (MODE == 2)
              atomicAdd(reinterpret_cast<unsigned long long*>(h + m * RS), (unsigned long long)(long long)rint(unit * v));
            else
              unsafeAtomicAdd(h + m * RS, (double)v);
          }
        };
        if constexpr (INC) {
          // Nothing below the first increment (everything below the grid counts at its first energy), everything
          // from the last one on; a lane takes energies in a row.
          int lo = direct && c0 == 0 ? 0 : c0 - 1;  // opaque, as in `point`
          asm volatile("" : "+v"(lo));
          const int full = (int)index(e[3], false, lo, a.ned);
          const int ja = min((int)index(e[0], true, lo, a.ned), full), ji = max(ja, c0), j1 = min(full, c1);
          const int per = (j1 - ji + (1 << lg)) >> lg, j0 = ji + sub * per, last = min(j0 + per - 1, j1);
          if (j0 > last) continue;
          NosVolumes v = nos_volumes(e);
          double prev[4] = {0.0, 0.0, 0.0, 0.0};
          if (j0 > ja) corner_nos(v, a.Vd, e0 + (j0 - 1 + joff) * a.ded, prev);
          for (int j = j0; j <= last; ++j) {
            double cur[4] = {a.Vd, a.Vd, a.Vd, a.Vd};
            float g[4];
            asm volatile("" : "+v"(v.e[0]), "+v"(v.e[1]), "+v"(v.e[2]), "+v"(v.e[3]));  // no doubles of them kept live
            if (j < full) corner_nos(v, a.Vd, e0 + (j + joff) * a.ded, cur);
            schedule_fence();
#pragma unroll
            for (int l = 0; l < 4; ++l) {
              g[l] = (float)(cur[l] - prev[l]);
              prev[l] = cur[l];
            }
            schedule_fence();
            put(j, g);
          }
        } else {
          tet_energies(e, a, max(c0, 0), c1, sub, 1 << lg, put);
        }
      }
    });
  };
  // The rows [lo, hi) of the histogram's `planes` + 1 planes, row r of energy row0 + r, into the result.
  auto flush = [&](int lo, int hi, int row0, int m0, int gm, int planes, int sexp) {
    asm volatile("" : "+s"(gm));  // its reciprocal is not kept over the groups of orbitals
    for_lanes((hi - lo) * gm, [&](int i) {
      const int q = gm == NORB ? i / NORB : i / gm, r = lo + q, m = i - q * gm;
      Acc v = hist[m * RS + r];
      for (int k = 1; k <= planes; ++k) v += hist[k * plane + m * RS + r];
      const int64_t at = (int64_t)(row0 + r) * NORB + m0 + m;
      if constexpr (MODE == 2) {
        const int dshift = exact_scale_exp(*a.gexp, a.lg_units) - sexp;
        long long fixed;
        if (dshift >= 0) fixed = (long long)((unsigned long long)v << dshift);
        else if (dshift > -63) fixed = (v + (1ll << (-dshift - 1))) >> (-dshift);
        else fixed = 0;
        if (fixed != 0) atomicAdd(&a.gacc[at], (unsigned long long)fixed);
      } else if constexpr (INC) {
        if (v != 0.0 && row0 + r >= a.shift)
          atomic_add_global(&a.dos[at - a.shift * NORB], (float)(v * a.out_scale));
      } else {
        if (v != 0.0) atomic_add_global(&a.dos[at], (float)v);
      }
    });
    __syncthreads();
  };

  const int lots = uniform(direct ? (J1 - J0 + RS) / RS : (NORB + group - 1) / group);
  for (int lot = 0; lot < lots; ++lot) {
    const int m0 = direct ? 0 : lot * group, m1 = min(m0 + group, NORB), gm = m1 - m0;
    const int c0 = direct ? J0 + lot * RS : J0, c1 = direct ? min(c0 + RS - 1, J1) : J1;
    int zero = 0;  // opaque, so that no register pair of it is kept
    asm volatile("" : "+v"(zero));
    for_lanes(copies * plane, [&](int i) { hist[i] = (Acc)zero; });
    int sexp = 0;
    if constexpr (MODE == 2) {
      // Fixed point: entries below 2^51, sums of every bin (below 2^gexp) below 2^62.
      sexp = 62 - *a.gexp;
      if (!none) {
        double dmax = 0.0;
        for_lanes(np, [&](int q) {
          point(q, m0, m1, c4, [&](int, int, const double D[4]) {
            dmax = fmax(dmax, fmax(fmax(fabs(D[0]), fabs(D[1])), fmax(fabs(D[2]), fabs(D[3]))));
          });
        });
        for (int o = 32; o > 0; o >>= 1) dmax = fmax(dmax, __shfl_xor(dmax, o));
        __syncthreads();
        if ((tid & 63) == 0) sh.dred[tid >> 6] = dmax;
        __syncthreads();
        for (int i = 0; i < NW; ++i) dmax = fmax(dmax, sh.dred[i]);
        int dexp;
        frexp(fmax(dmax, 1.0e-290), &dexp);  // dmax < 2^dexp
        sexp = min(51 - dexp, sexp);
      }
      sexp = uniform(sexp);
    }
    __syncthreads();
    const int spread = nq > kQueue / 8 ? copies - 1 : 0;  // planes for the sums energy by energy
    if (!none) {
      const double scale = MODE == 2 ? uniform(ldexp(c4, sexp)) : c4;
      for_lanes(np, [&](int q) {
        Acc* const mine = hist + (q & (copies - 1)) * plane;
        point(q, m0, m1, scale, [&](int m, int row, const double D[NE]) {
          Acc* h = &mine[(m - m0) * RS + row];
#pragma unroll
          for (int i = 0; i < NE; ++i) {
            if constexpr (MODE == 2) {
              constexpr double magic = 6755399441055744.0;  // 1.5 * 2^52: the sum's low bits are the rounded value
              const long long v = __double_as_longlong(D[i] + magic) - __double_as_longlong(magic);
              atomicAdd(reinterpret_cast<unsigned long long*>(&h[i]), (unsigned long long)v);
            } else {
              unsafeAtomicAdd(&h[i], D[i]);
            }
          }
        });
      });
      __syncthreads();
      running_sums(hist, gm, RS, plane, copies, rows, spread > 0);
      __syncthreads();
    }
    if (nq > 0) {  // the tetrahedra left out, onto the sums
      const bool all = direct || nq > kQueue;
      const int count = all ? 6 * ncubes : nq;
      int lg = all ? (c1 - c0 >= kLongRows) : 4;
      while (!all && lg > 0 && (count << lg) > NT) --lg;
      sum_tets(count, lg, all, m0, m1, c0, c1, spread, sexp);
      __syncthreads();
    }
    const int lo = max(-c0, 0);
    if (INC && lo > 0 && a.shift == 0) {  // increments below the grid count at its first energy
#pragma unroll 1
      for (int m = 0; m < gm; ++m)
        for_lanes(lo, [&](int r) {
          double v = 0.0;
          for (int k = 0; k <= spread; ++k) v += sh.hist[k * plane + m * RS + r];
          unsafeAtomicAdd(&sh.hist[m * RS + lo], v);
        });
      __syncthreads();
    }
    flush(lo, c1 - c0 + 1, c0, m0, gm, spread, sexp);
  }
}

template <int NORB, typename WT, int MODE>
__global__ __launch_bounds__(NTMAX, kWaves) void dos_forward_kernel(FwdArgs a) {
  // XCD-aware mapping: hardware dispatches block b to XCD b % 8; give each XCD a contiguous range.
  const int b = blockIdx.x;
  const int unit = (b % NXCD) * a.per_xcd + b / NXCD;
  if (unit >= a.nunits) return;
  if constexpr (MODE == 1) {
    __shared__ BoundShared<NORB> sh;
    bound_unit<NORB, WT>(a, unit, sh);
  } else {
    __shared__ SplineShared<NORB> sh;
    spline_unit<NORB, WT, MODE>(a, unit, sh);
  }
}

// ---------------------------------------------------------------------------------------------
// Batched forward: one launch over the flattened (item, band, tile) units of up to kMaxBatch problems with
// the same orbital count, a workgroup per unit.

template <int NORB, typename WT>
__global__ __launch_bounds__(NTMAX, kWaves) void dos_batched_kernel(BatchArgs b) {
  __shared__ SplineShared<NORB> sh;
  const int blk = blockIdx.x;
  const int u = (blk % NXCD) * b.per_xcd + blk / NXCD;  // each XCD a contiguous range of units
  if (u >= b.total) return;
  int i = 0;
  while (i + 1 < b.n && b.it[i + 1].unit_begin <= u) ++i;
  const BatchItem& it = b.it[i];
  FwdArgs a;
  a.eps = it.eps;
  a.w = it.w;
  a.w_scale = it.w_scale;
  a.dos = it.dos;
  a.n1 = it.n1;
  a.n2 = it.n2;
  a.n3 = it.n3;
  a.ne = it.ne;
  a.e0 = it.e0;
  a.de = it.de;
  a.inv_de = 1.0f / it.de;
  a.e0d = it.e0;
  a.ded = it.de;
  a.ned = it.ne;
  const double V = 1.0 / (24.0 * (double)it.n1 * it.n2 * it.n3);  // V_T / (4 V_G)
  a.V = (float)V;
  a.inv_ded = 1.0 / (double)it.de;
  a.c4 = 4.0 * V * a.inv_ded;
  a.t2 = it.t2;
  a.t3 = it.t3;
  a.s1 = it.s & 0xff;
  a.s2 = (it.s >> 8) & 0xff;
  a.s3 = it.s >> 16;
  a.r1 = it.r1;
  a.r2 = it.r2;
  a.r3 = it.r3;
  a.by_ntiles = it.by_ntiles;
  a.by_t2 = it.by_t2;
  a.by_t3 = it.by_t3;
  a.ntiles = it.ntiles;
  a.unit = step_unit(it.de);
  a.width = it.de * a.unit;
  a.degenerate = it.degenerate;
  spline_unit<NORB, WT, 0>(a, u - it.unit_begin, sh);
}

// Zero every item's DOS (blockIdx.y = item).
__global__ void batched_zero_kernel(BatchArgs b, int norb) {
  const BatchItem& it = b.it[blockIdx.y];
  const int64_t n = (int64_t)it.ne * norb;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    it.dos[i] = 0.0f;
}

template <int NORB, typename WT, int MODE>
void launch_fwd_type(const FwdArgs& a, int grid, hipStream_t s) {
  if (a.window)
    hipLaunchKernelGGL((dos_window_kernel<NORB, WT, MODE>), dim3(grid), dim3(kTileCubes), 0, s, a);
  else
    hipLaunchKernelGGL((dos_forward_kernel<NORB, WT, MODE>), dim3(grid), dim3(a.lanes), 0, s, a);
}
template <int NORB, int MODE>
hipError_t launch_fwd_mode(const FwdArgs& a, int grid, hipStream_t s) {
  if (a.wtype == TETRA_W_F16)
    launch_fwd_type<NORB, _Float16, MODE>(a, grid, s);
  else if (a.wtype == TETRA_W_C32)
    launch_fwd_type<NORB, float2, MODE>(a, grid, s);
  else
    launch_fwd_type<NORB, float, MODE>(a, grid, s);
  return hipGetLastError();
}

// dos = acc / S with S the common scale of mode 2 (all zero when no workgroup had anything to add).
__global__ void fixed_to_float_kernel(const unsigned long long* acc, const int* gexp, int lg_units, float* dos,
                                      int64_t n) {
  const int ge = *gexp;
  const double inv_S = ge == kNoBound ? 0.0 : ldexp(1.0, -exact_scale_exp(ge, lg_units));
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    dos[i] = (float)((double)(long long)acc[i] * inv_S);
}

}  // namespace

template <int NORB>
hipError_t launch_batched(const BatchArgs& b, int wtype, hipStream_t s) {
  hipLaunchKernelGGL(batched_zero_kernel, dim3(8, b.n), dim3(256), 0, s, b, NORB);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int grid = b.per_xcd * NXCD;
  if (wtype == TETRA_W_F16)
    hipLaunchKernelGGL((dos_batched_kernel<NORB, _Float16>), dim3(grid), dim3(b.lanes), 0, s, b);
  else if (wtype == TETRA_W_C32)
    hipLaunchKernelGGL((dos_batched_kernel<NORB, float2>), dim3(grid), dim3(b.lanes), 0, s, b);
  else
    hipLaunchKernelGGL((dos_batched_kernel<NORB, float>), dim3(grid), dim3(b.lanes), 0, s, b);
  return hipGetLastError();
}

template <int NORB>
hipError_t launch_fwd(const FwdArgs& a, int grid, hipStream_t s) {
  if (!a.gacc) return launch_fwd_mode<NORB, 0>(a, grid, s);
  hipError_t e = launch_fwd_mode<NORB, 1>(a, grid, s);
  if (e != hipSuccess) return e;
  e = launch_fwd_mode<NORB, 2>(a, grid, s);
  if (e != hipSuccess) return e;
  const int64_t n = (int64_t)a.ne * NORB;
  hipLaunchKernelGGL(fixed_to_float_kernel, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 4096)), dim3(256), 0, s,
                     a.gacc, a.gexp, a.lg_units, a.dos, n);
  return hipGetLastError();
}

}  // namespace tetra
