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
// Degenerate tetrahedra go energy by energy onto the sums, as in the forward; with weights that are not finite or energy
// ranges beyond the histogram all of them.
//
// 64^3 x 8 x 8 x 500 (9,830 pairs of a tile and two bands with something to add, 19 % of their tetrahedra left out):
// 0.73 ms, of it 0.15 workgroups that find no pair, 0.14 differences and words, 0.18 weights (16 loads per point,
// three times what the forward stages for its 8), 0.38 coefficients and contractions, 0.04 each deposits and sums. VALU
// busy for 0.60 of the cycles, the LDS for 0.37. Four simple cubic bands x 8 orbitals, 64^3 x 1000, the whole call: 1.82 ms
// with the loop over windows, 1.31 ms now (3.16 ms when tiles with many degenerate tetrahedra summed all of them energy
// by energy); layered bands 6.56, 4.59 (15.3) ms.
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
  int n1 = a.n1, n2s = a.n2, n3 = a.n3;
  asm volatile("" : "+s"(n1), "+s"(n2s), "+s"(n3));  // no copies in vector registers from one pair to the next
  auto grid_index = [&](int q, int s1, int s2, int s3) {
    int px, py, pz;
    split(q, px, py, pz);
    return ((int64_t)wrap(x0 + px + s1, n1) * n2s + wrap(y0 + py + s2, n2s)) * n3 + wrap(z0 + pz + s3, n3);
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
  double far = kFarKnot;  // opaque: the constant is not kept from one pair to the next
  asm volatile("" : "+v"(far));
  for_lanes(kKnotPad, [&](int i) { sh.u[i] = far; });
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
  const bool wide = !(rows_d + 6.0 <= (double)chi_spline_words<NORB>());
  const int base = wide ? 0 : uniform((int)floor(umin)), rows = wide ? 1 : uniform((int)rows_d);
  const int first = uniform((int)fmin(fmax(floor(umin), 0.0), a.ned));  // energy by energy
  const int last = uniform((int)fmin(ceil(umax), a.ned - 1.0));
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
  // The weights, and whether one of them is not finite.
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
    if (!(sum < 3.0e38f)) atomicOr(&sh.signs, 4);
  }
  __syncthreads();
  const int nq = uniform(sh.nq), signs = uniform(sh.signs);
  const bool finite = !(signs & 4), direct = wide || !finite;  // direct: every tetrahedron energy by energy

  int group = NORB, RS = (rows + 5) | 1, J0 = base, J1 = base + rows - 1;
  if (direct) {  // all orbitals, some energies at a time
    J0 = first;
    J1 = last;
    RS = (chi_spline_words<NORB>() / NORB - 2) | 1;
  }
  while ((RS * group | 1) > chi_spline_words<NORB>()) group = (group + 1) / 2;
  const int plane = RS * group | 1;  // odd: the copies of a bin in different banks
  const int copies = histogram_copies(plane, chi_spline_words<NORB>());

  // The `count` tetrahedra of the queue energy by energy, or all that take part and not in the spline form (count: all
  // there are), 2^lg lanes each: the energies [c0, c1] and orbitals [m0, m1) into rows from c0 on, lane i into plane
  // i & planes. Neighbouring lanes take tetrahedra that do not lie next to each other, as in the forward.
  auto sum_tets = [&](int count, int lg, bool all, int m0, int m1, int c0, int c1, int planes) {
    constexpr int G = NORB < 8 ? NORB : 8;  // orbitals whose weights a lane holds
    const int eighth = (count + 7) >> 3, area = tl.cx * cy, by_cx = small_inverse(tl.cx);
    for_lanes((all ? count : 8 * eighth) << lg, [&](int i) {
      const int k = i >> lg, sub = i & ((1 << lg) - 1);
      int t, ix, iy, iz;
      if (all) {
        t = (k >= ncubes) + (k >= 2 * ncubes) + (k >= 3 * ncubes) + (k >= 4 * ncubes) + (k >= 5 * ncubes);
        const int q = k - t * ncubes, z = small_div(small_div(q, by_cx), by_cy), r = q - z * area;
        ix = small_div(r, by_cy);
        iy = r - ix * cy;
        iz = z + ix + iy;
        iz -= small_div(iz, by_cz) * cz;
      } else {
        const int q = (k & 7) * eighth + (k >> 3);
        if (q >= count) return;
        const int it = sh.queue[q], cb = it / 6;
        t = it - 6 * cb;
        cube(cb, ix, iy, iz);
      }
      const uint32_t slots = tet_slots(t);
      float d[4];
      int pt[4];
      uint32_t side = 3u;
#pragma unroll
      for (int l = 0; l < 4; ++l) {
        const int s = (slots >> (4 * l)) & 7;
        pt[l] = (ix + (s & 1)) * PY + (iy + ((s >> 1) & 1)) * PZ + iz + (s >> 2);
        d[l] = sh.d[pt[l]];
        side &= sh.side[pt[l]];
      }
      // side 0: E_F cuts it or no transition (a corner without a finite energy has no side); both: flat
      const uint32_t word = (uint32_t)sh.word[(ix + 1) * CY + (iy + 1) * CZ + iz + 1] >> t;
      if (side == 0u || (!direct && !(word & ((side & 1u) ? 1u : 0x100u)))) return;
      sort4(d, pt);
      if (!(d[3] > d[0]) || !(d[3] > a.e0)) return;
      const float sign = (side & 1u) ? 1.0f : -1.0f;
      double* const h0 = sh.hist + (i & planes) * plane - c0;
#pragma unroll 1
      for (int mc = m0; mc < m1; mc += G) {
        float wt[4][G];
#pragma unroll
        for (int m = 0; m < G; ++m) {
          const int at = min(mc + m, m1 - 1);
#pragma unroll
          for (int l = 0; l < 4; ++l) wt[l][m] = sign * sh.w[at * NP + pt[l]];
          if (!finite) {  // a weight that is no number adds nothing
            const float sum = (wt[0][m] + wt[1][m]) + (wt[2][m] + wt[3][m]);
#pragma unroll
            for (int l = 0; l < 4; ++l) wt[l][m] = sum == sum ? wt[l][m] : 0.0f;
          }
        }
        tet_energies(d, a, max(c0, 0), c1, sub, 1 << lg, [&](int j, const float g[4]) {
          double* h = h0 + (mc - m0) * RS + j;
#pragma unroll
          for (int m = 0; m < G; ++m) {
            if (mc + m >= m1) continue;
            const float v = g[0] * wt[0][m] + g[1] * wt[1][m] + g[2] * wt[2][m] + g[3] * wt[3][m];
            unsafeAtomicAdd(h + m * RS, (double)v);
          }
        });
      }
    });
  };

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

  const int lots = uniform(direct ? (J1 - J0 + RS) / RS : (NORB + group - 1) / group);
  for (int lot = 0; lot < lots; ++lot) {
    const int m0 = direct ? 0 : lot * group, m1 = min(m0 + group, NORB), gm = m1 - m0;
    const int c0 = direct ? J0 + lot * RS : J0, c1 = direct ? min(c0 + RS - 1, J1) : J1;
    int zero = 0;  // opaque, so that no register pair of it is kept
    asm volatile("" : "+v"(zero));
    for_lanes(copies * plane, [&](int i) { sh.hist[i] = (double)zero; });
    __syncthreads();
    const int spread = nq > kQueue / 8 ? copies - 1 : 0;  // planes for the sums energy by energy
    if (!direct) {
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
      __syncthreads();
      running_sums(sh.hist, gm, RS, plane, copies, rows, spread > 0);
      __syncthreads();
    }
    if (direct || nq > 0) {  // the tetrahedra left out, onto the sums
      const bool all = direct || nq > kQueue;
      const int count = all ? 6 * ncubes : nq;
      int lg = all ? (c1 - c0 >= kLongRows) : 4;
      while (!all && lg > 0 && (count << lg) > NT) --lg;
      sum_tets(count, lg, all, m0, m1, c0, c1, spread);
      __syncthreads();
    }
    const int lo = max(-c0, 0);
    int gd = gm;
    asm volatile("" : "+s"(gd));  // its reciprocal is not kept over the groups of orbitals
    for_lanes((c1 - c0 + 1 - lo) * gm, [&](int i) {
      const int r0 = gm == NORB ? i / NORB : i / gd, r = lo + r0, m = i - r0 * gm;
      double v = sh.hist[m * RS + r];
      for (int k = 1; k <= spread; ++k) v += sh.hist[k * plane + m * RS + r];
      if (v != 0.0) atomic_add_global(&a.dos[(int64_t)(c0 + r) * NORB + m0 + m], (float)v);
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
