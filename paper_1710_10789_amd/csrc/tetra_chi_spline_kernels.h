// First pass of the susceptibility (tetra_chi_device.h): the tetrahedra that are occupied in one band and
// empty in the other at every corner, in the spline form (tetra_spline.h), on gfx950.
//
// There the spectral weight is the DOS of the difference energy d = eps_n'(k + q) - eps_n(k) with the product
// weights W_m = b_mn(k) b_mn'(k + q): +1 times it where n is occupied, -1 times it where n' is. One workgroup
// per (tile of at most 8 x 8 x 8 cubes, band pair), units tile-major, and the forward's steps: d in grid
// steps as knots, one lane per grid point for the truncated powers of all of the tile's tetrahedra around
// it, FP64 histogram of fourth differences, running sums. What is left out here: tetrahedra that E_F cuts in
// a band (the clipping kernel's), those off the energy grid, degenerate ones (through a queue). The two signs
// are two sweeps over the points (a unit with both is rare: the signs held beside the masks of one sweep took
// more registers than there are). A cube has a word for each: which of its six take no part (bits 0-5, for the
// negative ones 8-13), whether any does (bit 6 or 14); a point forms its mask from the eight cubes around it.
// Tiles with weights that are not finite, more degenerate tetrahedra than the queue holds or energy ranges
// beyond the histogram: a lane per tetrahedron, energy by energy into the histogram, some energies at a time.
//
// 64^3 x 8 x 8 x 500 (9,830 pairs of a tile and two bands with something to add, 19 % of their tetrahedra left out):
// 0.71 ms, of it 0.15 workgroups that find no pair, 0.14 differences and words, 0.18 weights (16 loads per point,
// three times what the forward stages for its 8), 0.38 coefficients and contractions, 0.04 each deposits and sums.
// No kernel here may spill vector registers (the compiler has placed such stores behind a loop's exit with no lane
// active).
#pragma once

#include "tetra_chi_args.h"
#include "tetra_chi_device.h"
#include "tetra_spline_tile.h"
#include "tetra_weights.h"

namespace tetra {

namespace {

constexpr int CZ = kSide + 2, CY = CZ * CZ;  // strides of the cubes' words, one empty cube around the tile

template <int NORB>
struct ChiSplineFixed {
  double u[kKnotPad];
  float d[NP];  // eps' - eps; not a number where either is not finite
  float wlo[kWeightPad];
  float w[NP * NORB];
  float whi[kWeightPad];
  unsigned short word[CZ * CY];
  unsigned char side[NP];  // bit 0: n occupied and n' empty at the point; bit 1: the reverse
  unsigned short queue[kQueue];
  float red[2 * NWMAX];
  int nq, signs;
};
template <int NORB>
constexpr int chi_spline_words() { return (kLdsBytes - 64 - (int)sizeof(ChiSplineFixed<NORB>)) / 8; }
template <int NORB>
struct ChiSplineShared : ChiSplineFixed<NORB> {
  double hist[chi_spline_words<NORB>()];
};

// The bands n' = n0 + bit, of 64, with which band n can contribute over the tile by the table of energy ranges
// (all of them without one). Every wave by itself, a lane per band.
__device__ __forceinline__ uint64_t live_bands(const ChiSplineArgs& c, const Tile& t, int n, int n0) {
  int lane = threadIdx.x;
  asm volatile("" : "+v"(lane));
  const int n2 = n0 + (lane & 63);
  bool live = n2 < c.nb;
  if (live && c.ranges) {
    const int X0 = t.x0 / c.TX, Y0 = t.y0 / c.TY, Z0 = t.z0 / c.TZ;
    const int X1 = (t.x0 + t.cx - 1) / c.TX, Y1 = (t.y0 + t.cy - 1) / c.TY, Z1 = (t.z0 + t.cz - 1) / c.TZ;
    float2 rk = make_float2(__builtin_huge_valf(), -__builtin_huge_valf()), rq = rk;
    for (int x = X0; x <= X1; ++x)
      for (int y = Y0; y <= Y1; ++y)
        for (int z = Z0; z <= Z1; ++z) {
          const int at = (x * c.u2 + y) * c.u3 + z;
          const float2 a = c.ranges[(int64_t)n * c.ut + at], b = c.ranges[(int64_t)(c.nb + n2) * c.ut + at];
          rk = make_float2(fminf(rk.x, a.x), fmaxf(rk.y, a.y));
          rq = make_float2(fminf(rq.x, b.x), fmaxf(rq.y, b.y));
        }
    live = rk.x <= rk.y && rq.x <= rq.y &&
           (region_possible(0, rk.x, rk.y, rq.x, rq.y, c.ef) || region_possible(1, rk.x, rk.y, rq.x, rq.y, c.ef));
    int K0, K1;
    range_window(rq.x - rk.y, rq.y - rk.x, c.f.e0, c.f.inv_de, c.f.ne, K0, K1);
    live = live && K0 <= K1;
  }
  return __ballot(live);
}

// The pair of bands (n, n2) over a tile; every lane of the workgroup calls it.
template <int NORB, typename WT>
__device__ __forceinline__ void chi_spline_unit(const ChiSplineArgs& c, const Tile& tl, int n, int n2,
                                                ChiSplineShared<NORB>& sh) {
  const FwdArgs& a = c.f;
  const int x0 = tl.x0, y0 = tl.y0, z0 = tl.z0, cy = tl.cy, cz = tl.cz;
  const int qy = cy + 1, qz = cz + 1, np = (tl.cx + 1) * qy * qz, ncubes = tl.cx * cy * cz;
  const int by_qz = small_inverse(qz), by_qy = small_inverse(qy), by_cz = small_inverse(cz), by_cy = small_inverse(cy);
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));  // nothing formed from it is kept live from one pair to the next
  const int NT = blockDim.x, NW = NT >> 6;
  const int64_t nk = (int64_t)a.n1 * a.n2 * a.n3;
  const float *eps_n = a.eps + (int64_t)n * nk, *eps_p = a.eps + (int64_t)n2 * nk;
  const double e0 = a.e0d, inv_de = a.inv_ded;
  auto split = [&](int q, int& px, int& py, int& pz) {
    const int r = small_div(q, by_qz);
    pz = q - r * qz;
    px = small_div(r, by_qy);
    py = r - px * qy;
  };
  auto grid_index = [&](int q, int s1, int s2, int s3) {
    int px, py, pz;
    split(q, px, py, pz);
    return ((int64_t)wrap(x0 + px + s1, a.n1) * a.n2 + wrap(y0 + py + s2, a.n2)) * a.n3 + wrap(z0 + pz + s3, a.n3);
  };

  // The differences and the sides of E_F; the loads of a lane's first two points in flight while the LDS is
  // prepared.
  float ahead_e[2], ahead_ep[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int q = tid + i * NT;
    if (q < np) {
      ahead_e[i] = eps_n[grid_index(q, 0, 0, 0)];
      ahead_ep[i] = eps_p[grid_index(q, c.q1, c.q2, c.q3)];
    }
  }
  for_lanes(kKnotPad, [&](int i) { sh.u[i] = kFarKnot; });
  for_lanes(kWeightPad, [&](int i) { sh.wlo[i] = sh.whi[i] = 0.0f; });
  for_lanes(CZ * CY, [&](int i) { sh.word[i] = 0; });
  if (np < NP) {  // every word a neighbour offset can reach holds a finite value
    for_lanes(NP * NORB, [&](int i) { sh.w[i] = 0.0f; });
  }
  if (tid == 0) sh.nq = sh.signs = 0;
  __syncthreads();
  auto stage = [&](int q, float e, float ep) {
    int px, py, pz;
    split(q, px, py, pz);
    const int p = px * PY + py * PZ + pz;
    const bool finite = __builtin_isfinite(e) && __builtin_isfinite(ep);
    const float d = ep - e;
    sh.d[p] = finite ? d : __builtin_nanf("");
    sh.side[p] = finite ? (unsigned char)((e <= c.ef && ep >= c.ef) | ((e >= c.ef && ep <= c.ef) << 1)) : 0;
    if (finite) sh.u[kKnotMargin + px * SY + py * SZ + pz] = ((double)d - e0) * inv_de;
  };
#pragma unroll
  for (int i = 0; i < 2; ++i)
    if (tid + i * NT < np) stage(tid + i * NT, ahead_e[i], ahead_ep[i]);
  for (int q0 = 2 * NT; q0 < np; q0 += NT) {  // only tiles one cube thick have so many points per lane
    const int q = q0 + tid;
    if (q < np) stage(q, eps_n[grid_index(q, 0, 0, 0)], eps_p[grid_index(q, c.q1, c.q2, c.q3)]);
  }
  __syncthreads();

  // A cube's tetrahedra: which take part (whole, not flat, not off the energy grid) and which of them count
  // negatively; d of the corners. Corners 2 and 5 belong to all six of Table I, the other two run around them.
  const float elast = (float)(e0 + (a.ned - 1.0) * a.ded);
  constexpr int I[6][2] = {{0, 1}, {1, 3}, {0, 4}, {3, 7}, {4, 6}, {6, 7}};
  auto cube = [&](int i, int& ix, int& iy, int& iz) {
    const int r = small_div(i, by_cz);
    iz = i - r * cz;
    ix = small_div(r, by_cy);
    iy = r - ix * cy;
  };
  auto cube_word = [&](int i) -> unsigned short& {
    int ix, iy, iz;
    cube(i, ix, iy, iz);
    return sh.word[(ix + 1) * CY + (iy + 1) * CZ + iz + 1];
  };
  auto analyse = [&](int i, float d[8], uint32_t& taken, uint32_t& minus) {
    int ix, iy, iz;
    cube(i, ix, iy, iz);
    const int p0 = ix * PY + iy * PZ + iz;
    uint32_t m0 = 0u, m1 = 0u;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int p = p0 + (s & 1) * PY + ((s >> 1) & 1) * PZ + (s >> 2);
      d[s] = sh.d[p];
      m0 |= (uint32_t)(sh.side[p] & 1) << s;
      m1 |= (uint32_t)(sh.side[p] >> 1) << s;
    }
    taken = minus = 0u;
    const float lo = fminf(d[2], d[5]), hi = fmaxf(d[2], d[5]);
#pragma unroll
    for (int t = 0; t < 6; ++t) {
      const uint32_t K = 1u << 2 | 1u << 5 | 1u << I[t][0] | 1u << I[t][1];
      const float dmin = fminf(lo, fminf(d[I[t][0]], d[I[t][1]])), dmax = fmaxf(hi, fmaxf(d[I[t][0]], d[I[t][1]]));
      const bool plus = (m0 & K) == K, in = (plus || (m1 & K) == K) && dmax > dmin && dmax > a.e0 && dmin <= elast;
      taken |= (uint32_t)in << t;
      minus |= (uint32_t)(in && !plus) << t;
    }
  };
  // The lane's cube (no tile has more cubes than lanes); range of d over its tetrahedra that take part.
  float lmin = __builtin_huge_valf(), lmax = -__builtin_huge_valf();
  float d8[8];
  uint32_t taken = 0u, minus = 0u;
  if (tid < ncubes) {
    analyse(tid, d8, taken, minus);
#pragma unroll
    for (int t = 0; t < 6; ++t)
      if ((taken >> t) & 1u) {
        lmin = fminf(lmin, fminf(fminf(d8[2], d8[5]), fminf(d8[I[t][0]], d8[I[t][1]])));
        lmax = fmaxf(lmax, fmaxf(fmaxf(d8[2], d8[5]), fmaxf(d8[I[t][0]], d8[I[t][1]])));
      }
  }
  lmin = wave_min(lmin);
  lmax = wave_max(lmax);
  if ((tid & 63) == 0) {
    sh.red[tid >> 6] = lmin;
    sh.red[NW + (tid >> 6)] = lmax;
  }
  __syncthreads();
  float dmin = sh.red[0], dmax = sh.red[NW];
  for (int i = 1; i < NW; ++i) {
    dmin = fminf(dmin, sh.red[i]);
    dmax = fmaxf(dmax, sh.red[NW + i]);
  }
  dmin = uniform(dmin);
  dmax = uniform(dmax);
  if (!(dmin <= dmax)) return;  // nothing takes part

  // Rows of the sums: from the first grid energy at or above the lowest knot to the last one below the highest.
  const double umin = ((double)dmin - e0) * inv_de, umax = ((double)dmax - e0) * inv_de;
  const double rows_d = fmin(ceil(umax), a.ned) - floor(umin);
  bool direct = !(rows_d + 6.0 <= (double)chi_spline_words<NORB>());
  const int base = direct ? 0 : uniform((int)floor(umin)), rows = direct ? 1 : uniform((int)rows_d);
  const int first = uniform((int)fmin(fmax(floor(umin), 0.0), a.ned));  // energy by energy
  const int last = uniform((int)fmin(ceil(umax), (a.ned - 1.0)));
  const float J = (float)rows, limit = a.degenerate * J * J * J;

  // The cube's word; degenerate tetrahedra into the queue.
  if (tid < ncubes) {
    const uint32_t plus = taken & ~minus;
    uint32_t bits = (plus ? 0x40u : 0u) | (minus ? 0x4000u : 0u) | (~plus & 0x3fu) | (~minus & 0x3fu) << 8;
    if (taken) atomicOr(&sh.signs, (int)(plus != 0u) | (int)(minus != 0u) << 1);
    const float lo = fminf(d8[2], d8[5]) * a.unit, hi = fmaxf(d8[2], d8[5]) * a.unit;
#pragma unroll
    for (int t = 0; t < 6; ++t) {
      const float x = d8[I[t][0]] * a.unit, y = d8[I[t][1]] * a.unit;
      if (!(spline_gap(lo, hi, fminf(x, y), fmaxf(x, y), a.width) >= limit) && ((taken >> t) & 1u)) {
        const int at = atomicAdd(&sh.nq, 1);
        if (at < kQueue) sh.queue[at] = (unsigned short)(tid * 6 + t);
        bits |= 0x101u << t;
      }
    }
    cube_word(tid) = (unsigned short)bits;
  }
  // The weights. One that is not finite counts as too many degenerate tetrahedra: energy by energy.
  {
    const WT* w_n = static_cast<const WT*>(a.w) + (int64_t)n * NORB * nk;
    const WT* w_p = static_cast<const WT*>(a.w) + (int64_t)n2 * NORB * nk;
    const float sc_n = a.w_scale ? a.w_scale[n] : 1.0f, sc_p = a.w_scale ? a.w_scale[n2] : 1.0f;
    float sum = 0.0f;
    for_lanes(np, [&](int q) {
      const int64_t k = grid_index(q, 0, 0, 0), kq = grid_index(q, c.q1, c.q2, c.q3);
      int px, py, pz;
      split(q, px, py, pz);
      float* w = &sh.w[px * PY + py * PZ + pz];
      WT b[NORB], b2[NORB];  // all in flight
#pragma unroll
      for (int m = 0; m < NORB; ++m) b[m] = w_n[(int64_t)m * nk + k];
#pragma unroll
      for (int m = 0; m < NORB; ++m) b2[m] = w_p[(int64_t)m * nk + kq];
#pragma unroll
      for (int m = 0; m < NORB; ++m) {
        const float W = weight_value(b[m], sc_n) * weight_value(b2[m], sc_p);
        w[m * NP] = W;
        sum += fabsf(W) * 0x1p-20f;
      }
    });
    if (!(sum < 3.0e38f)) atomicAdd(&sh.nq, kQueue + 1);
  }
  __syncthreads();
  const int nq = uniform(sh.nq), signs = uniform(sh.signs);
  direct = direct || nq > kQueue;

  // A tetrahedron's corners sorted by d, with their points.
  auto corners = [&](int i, int t, float d[4], int pt[4]) {
    int ix, iy, iz;
    cube(i, ix, iy, iz);
    const uint32_t slots = tet_slots(t);
#pragma unroll
    for (int l = 0; l < 4; ++l) {
      const int s = (slots >> (4 * l)) & 7;
      pt[l] = (ix + (s & 1)) * PY + (iy + ((s >> 1) & 1)) * PZ + iz + (s >> 2);
      d[l] = sh.d[pt[l]];
    }
    sort4(d, pt);
  };

  if (direct) {
    if (tid < ncubes) {
      float dc[8];
      uint32_t in, neg;
      analyse(tid, dc, in, neg);
      cube_word(tid) = (unsigned short)(in | neg << 8);
    }
    constexpr int chunk = chi_spline_words<NORB>() / NORB;
    for (int c0 = first; c0 <= last; c0 += chunk) {
      const int c1 = min(c0 + chunk - 1, last), L = c1 - c0 + 1;
      __syncthreads();
      for_lanes(chunk * NORB, [&](int i) { sh.hist[i] = 0.0; });
      __syncthreads();
      constexpr int G = NORB < 8 ? NORB : 8;  // orbitals whose weights a lane holds
#pragma unroll 1
      for (int m0 = 0; m0 < NORB; m0 += G)
      for_lanes(ncubes * 6, [&](int i6) {
        const int ic = i6 / 6, t = i6 - 6 * ic;
        const uint32_t bits = (uint32_t)cube_word(ic) >> t;
        if (!(bits & 1u)) return;
        float d[4], wt[4][G];
        int pt[4];
        corners(ic, t, d, pt);
        const float sign = (bits & 0x100u) ? -1.0f : 1.0f;
#pragma unroll
        for (int l = 0; l < 4; ++l)
#pragma unroll
          for (int m = 0; m < G; ++m) wt[l][m] = m0 + m < NORB ? sign * sh.w[(m0 + m) * NP + pt[l]] : 0.0f;
        tet_energies(d, a, c0, c1, 0, 1, [&](int j, const float g[4]) {
          double* h = &sh.hist[m0 * chunk + j - c0];
#pragma unroll
          for (int m = 0; m < G; ++m)
            if (m0 + m < NORB) {
              const float v = g[0] * wt[0][m] + g[1] * wt[1][m] + g[2] * wt[2][m] + g[3] * wt[3][m];
              if (v == v) unsafeAtomicAdd(&h[m * chunk], (double)v);  // a weight that is no number adds nothing
            }
        });
      });
      __syncthreads();
      for_lanes(L * NORB, [&](int i) {
        const int r = i / NORB, m = i - r * NORB;
        const double v = sh.hist[m * chunk + r];
        if (v != 0.0) atomic_add_global(&a.dos[(int64_t)(c0 + r) * NORB + m], (float)v);
      });
    }
    return;
  }

  const int RS = (rows + 5) | 1;
  int group = NORB;
  while ((RS * group | 1) > chi_spline_words<NORB>()) group = (group + 1) / 2;
  const int plane = RS * group | 1;  // odd: the copies of a bin in different banks
  const int copies = histogram_copies(plane, chi_spline_words<NORB>());

  auto point = [&](int q, int sign, int m0, int m1, auto&& act) {
    int px, py, pz;
    split(q, px, py, pz);
    const double* up = &sh.u[kKnotMargin + px * SY + py * SZ + pz];
    const double u0 = up[0], ju = ceil(u0);
    // no cube with tetrahedra that take part, above the last row or below the first one (then none of them is
    // this point's) or not finite
    const unsigned short* word = &sh.word[px * CY + py * CZ + pz];  // the cube before the point on every axis
    uint32_t wd[8], any = 0u;  // by the point's corner slot in the cube
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      wd[s] = word[(1 - (s & 1)) * CY + (1 - ((s >> 1) & 1)) * CZ + 1 - (s >> 2)];
      any |= wd[s];
    }
    // the row numbers opaque, so that no double of them is kept live over the whole unit
    int b = base;
    asm volatile("" : "+v"(b));
    const double jr = ju - b;
    if (!((any >> (8 * sign)) & 0x40u) || !(jr < (double)rows) || jr < 0.0) return;
    const bool masks = __any(((any >> (8 * sign)) & 0x3fu) != 0u);
    uint32_t skip = 0u;
    if (masks) {
#pragma unroll
      for (int t = 0; t < 6; ++t)
#pragma unroll
        for (int l = 0; l < 4; ++l)
          skip |= ((wd[(tet_slots(t) >> (4 * l)) & 7] >> (8 * sign + t)) & 1u) << (4 * t + l);
    }
    schedule_fence();
    double M[kNeighbours];
    knot_reciprocals(up, u0, M);
    const int p = px * PY + py * PZ + pz;
    const double T = masks ? knot_coefs_skip(M, skip) : knot_coefs(M);
    double Ms = 0.0;
#pragma unroll
    for (int u = 0; u < kNeighbours; ++u) Ms += M[u];
    double N[4], n[4];
    knot_differences(ju - u0, N, n);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      N[i] *= sign ? -a.c4 : a.c4;
      n[i] *= (sign ? -a.c4 : a.c4) * T;
    }
    const int row = (int)jr;
#pragma unroll 2
    for (int m = m0; m < m1; ++m) {
      const float* w = sh.w + m * NP + p;
      const double bp = w[0], Q = knot_contract(M, Ms, w);
      double D[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) D[i] = __builtin_fma(Q, N[i], bp * n[i]);
      act(m, row, D);
    }
  };

  for (int m0 = 0; m0 < NORB; m0 += group) {
    const int m1 = min(m0 + group, NORB), gm = m1 - m0;
    for_lanes(copies * plane, [&](int i) { sh.hist[i] = 0.0; });
    __syncthreads();
    for (int sign = 0; sign < 2; ++sign) {
      if (!((signs >> sign) & 1)) continue;
      for_lanes(np, [&](int q) {
        double* const mine = sh.hist + (q & (copies - 1)) * plane;
        point(q, sign, m0, m1, [&](int m, int row, const double D[4]) {
          double* h = &mine[(m - m0) * RS + row];
#pragma unroll
          for (int i = 0; i < 4; ++i) unsafeAtomicAdd(&h[i], D[i]);
        });
      });
    }
    // degenerate tetrahedra, 16 lanes each: the fourth differences of the value at one energy
    for_lanes(16 * nq, [&](int i16) {
      const int item = sh.queue[i16 >> 4], i = item / 6, t = item - 6 * i;
      float d[4];
      int pt[4];
      corners(i, t, d, pt);
      const bool minus = !(sh.side[pt[0]] & sh.side[pt[1]] & sh.side[pt[2]] & sh.side[pt[3]] & 1);
      tet_energies(d, a, 0, a.ne - 1, i16 & 15, 16, [&](int j, const float g[4]) {
#pragma unroll 1
        for (int m = m0; m < m1; ++m) {
          const float* w = sh.w + m * NP;
          const double v = (double)g[0] * w[pt[0]] + (double)g[1] * w[pt[1]] + (double)g[2] * w[pt[2]] +
                           (double)g[3] * w[pt[3]], x = minus ? -v : v;
          double* h = &sh.hist[(m - m0) * RS + j - base];
          unsafeAtomicAdd(h, x);
          unsafeAtomicAdd(h + 1, -4.0 * x);
          unsafeAtomicAdd(h + 2, 6.0 * x);
          unsafeAtomicAdd(h + 3, -4.0 * x);
          unsafeAtomicAdd(h + 4, x);
        }
      });
    }, true);
    __syncthreads();
    running_sums(sh.hist, gm, RS, plane, copies, rows);
    __syncthreads();
    const int lo = max(-base, 0);
    for_lanes((rows - lo) * gm, [&](int i) {
      const int r0 = gm == NORB ? i / NORB : i / gm, r = lo + r0, m = i - r0 * gm;
      const double v = sh.hist[m * RS + r];
      if (v != 0.0) atomic_add_global(&a.dos[(int64_t)(base + r) * NORB + m0 + m], (float)v);
    });
    __syncthreads();
  }
}

// A workgroup takes every parts-th of the bands n' that are live with its band n over its tile: the others, most of
// them, cost no workgroup (0.98 ms with a workgroup per pair, 0.71 ms with three per (tile, n)).
template <int NORB, typename WT>
__global__ __launch_bounds__(NTMAX, kWaves) void chi_spline_kernel(ChiSplineArgs c) {
  __shared__ ChiSplineShared<NORB> sh;
  const int blk = blockIdx.x;
  const int unit = (blk % NXCD) * c.per_xcd + blk / NXCD;  // tile-major: the tile's points stay in the XCD's L2
  if (unit >= c.nunits) return;
  const int64_t u = c.first + unit;
  const int per_tile = c.nb * c.parts, tile = (int)(u / per_tile), r = (int)(u - (int64_t)tile * per_tile);
  const int n = r / c.parts, part = r - n * c.parts;
  int none;
  const Tile tl = unit_tile(c.f, tile, none);
  int k = 0;
  for (int n0 = 0; n0 < c.nb; n0 += 64)
    for (uint64_t live = live_bands(c, tl, n, n0); live; live &= live - 1) {
      if (k++ % c.parts != part) continue;
      chi_spline_unit<NORB, WT>(c, tl, n, n0 + __builtin_ctzll(live), sh);
      __syncthreads();
    }
}

}  // namespace

template <int NORB>
hipError_t launch_chi_spline(const ChiSplineArgs& a, hipStream_t s) {
  const int grid = a.per_xcd * NXCD;
  const dim3 lanes(a.f.lanes < 256 ? 256 : a.f.lanes);  // small and flat tiles: more lanes than cubes for the rest
  if (a.f.wtype == TETRA_W_F16)
    hipLaunchKernelGGL((chi_spline_kernel<NORB, _Float16>), dim3(grid), lanes, 0, s, a);
  else if (a.f.wtype == TETRA_W_C32)
    hipLaunchKernelGGL((chi_spline_kernel<NORB, float2>), dim3(grid), lanes, 0, s, a);
  else
    hipLaunchKernelGGL((chi_spline_kernel<NORB, float>), dim3(grid), lanes, 0, s, a);
  return hipGetLastError();
}

}  // namespace tetra
