// Forward kernels: orbital-resolved tetrahedron DOS on gfx950.
//
// Sum of eq. (tetracontriborbitalresolved) over the tetrahedra and bands of a periodic k-grid
// (eq. tetmethoorbitalresolved, Guterding & Jeschke, arXiv:1710.10789, Sec. II.C), with the
// tetrahedra of Table I.
//
// Work decomposition: one workgroup per (tile of at most 8 x 8 x 8 cubes, band). The tile's grid points
// (9 x 9 x 9: 1.42 points per cube; 4 x 4 x 16 cubes have 1.66) are staged once in LDS, energies and
// orbital weights. Then, two ways:
//  * the spline form (tetra_spline.h), nearly always: one lane per grid point forms the coefficients of the
//    point's truncated powers from all tetrahedra of the tile around it and adds four entries per orbital to
//    an LDS histogram of fourth differences (FP64 atomics, 8 lane-adds per clock and CU against 0.3 for FP32
//    ones); four running sums down the histogram give the tile's DOS. The work per tile does not depend on
//    the energy windows: 64^3 x 8 x 8 x 1000 took 0.32 ms with a loop over every tetrahedron's window and
//    takes 0.167 ms; 24^3 x 8 x 8 x 4096, with windows of 75 energies, 0.04 ms. Bound by FP64 issue
//    (about 560 instructions per point, 516 of them FP64) and the LDS (120 weight reads and 32 atomics per
//    point of 8 orbitals) in about equal parts.
//    Tetrahedra with nearly equal corner energies go through a queue, energy by energy.
//  * the general form: one lane per cube, a five-comparator sort of the corner energies and a loop over each
//    tetrahedron's energies. For the tile-bands that the spline form is not for: energy ranges beyond its
//    histogram (thousands of energies), more than kQueue degenerate tetrahedra (a band without dispersion
//    along an axis, a grid with a single point along one), weights that are not finite.
//    The LDS histogram there holds 64-bit fixed-point integers (LDS FP32 atomics are slow): every
//    contribution is non-negative (a corner weight is the section integral of a barycentric coordinate) and
//    a tetrahedron's point DOS never exceeds 3 V_T/(V_G E41), so with bmax = max |b| of the tile, a bound
//    B = sum 12 V bmax / E41 over the tetrahedra with a non-empty window bounds every bin's |sum| and fixes
//    a power-of-two scale S with B*S <= 2^62 (two's complement, so signed weights work too). When the
//    tile's weights are non-negative and its bound is not dominated by narrow tetrahedra (E41 < 2 de, whose
//    spikes would make B loose), two orbitals share one 64-bit atomic as two 32-bit fields with
//    B*S <= 2^30 (no carry between fields).
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

namespace tetra {

namespace {

// Words of the general form's LDS histogram.
template <int NORB>
constexpr int fwd_hist_words() { return NORB <= 8 ? 1280 : NORB == 16 ? 1344 : 2048; }
// Common fixed point of the exact mode: with E the largest bound exponent of any workgroup (each
// workgroup's bins sum to at most 2^E in magnitude) and L = ceil(log2(workgroups)), the total of any
// bin is below 2^(E + L), so the scale 2^(62 - E - L) keeps every partial and total sum of the
// 64-bit two's-complement accumulator in range.
__device__ __forceinline__ int exact_scale_exp(int gexp, int lg_units) { return 62 - gexp - lg_units; }

// Shared memory and body of the general form.
template <int NORB>
struct GeneralShared {
  float eps[NP];
  float w[NP * NORB];
  unsigned long long hist[fwd_hist_words<NORB>()];
  float red[4 * NWMAX];
};

// One work unit (tile, band) of the forward pass in the general form; every lane of the workgroup calls it.
// MODE 0: DOS with per-workgroup scales, flushed with float atomics;
// 1: only the workgroup's bound exponent, into *gexp (atomicMax: independent of the order);
// 2: DOS with per-workgroup scales as in mode 0; each bin's exact per-workgroup sum is rounded once
//    to the common fixed point fixed by *gexp and added to gacc with a 64-bit integer atomic. Both
//    steps are independent of the order in which workgroups run, so the result is bitwise
//    reproducible.
template <int NORB, typename WT, int MODE>
__device__ __forceinline__ void general_unit(const FwdArgs& a, int unit, GeneralShared<NORB>& sh) {
  constexpr int NPAIR = (NORB + 1) / 2;
  // Histogram rows (one per orbital pair in the packed form, one per orbital in the wide form) have a
  // fixed, odd stride in 64-bit words: the row offsets of a deposit are immediates, and the flush
  // reads across rows without bank conflicts.
  constexpr int HCAP = fwd_hist_words<NORB>();
  constexpr int RSP = (HCAP / NPAIR - 1) | 1, RSW = (HCAP / NORB - 1) | 1;
  float* const s_eps = sh.eps;
  float* const s_w = sh.w;
  unsigned long long* const s_hist = sh.hist;
  float* const s_red = sh.red;

  int band;
  const Tile tl = unit_tile(a, unit, band);
  const int x0 = tl.x0, y0 = tl.y0, z0 = tl.z0;
  const int qy = tl.cy + 1, qz = tl.cz + 1, np = (tl.cx + 1) * qy * qz, ncubes = tl.cx * tl.cy * tl.cz;
  const int by_qz = small_inverse(qz), by_qy = small_inverse(qy);
  const int tid = threadIdx.x, NT = blockDim.x, NW = NT >> 6;
  const int64_t nk = (int64_t)a.n1 * a.n2 * a.n3;
  const float* eps_n = a.eps + (int64_t)band * nk;
  const WT* w_n = static_cast<const WT*>(a.w) + (int64_t)band * NORB * nk;
  const float wscale = a.w_scale ? a.w_scale[band] : 1.0f;

  // Stage the tile's grid points (periodic wrap) and find their energy range.
  float lmin = __builtin_huge_valf(), lmax = -__builtin_huge_valf(), lbmax = 0.0f, lbmin = 0.0f;
  for (int q = tid; q < np; q += NT) {
    const int r = small_div(q, by_qz), pz = q - r * qz, px = small_div(r, by_qy), py = r - px * qy;
    const int p = px * PY + py * PZ + pz;
    const int64_t k = ((int64_t)wrap(x0 + px, a.n1) * a.n2 + wrap(y0 + py, a.n2)) * a.n3 + wrap(z0 + pz, a.n3);
    const float e = eps_n[k];
    s_eps[p] = e;
    if (__builtin_isfinite(e)) {
      lmin = fminf(lmin, e);
      lmax = fmaxf(lmax, e);
    }
#pragma unroll
    for (int m = 0; m < NORB; ++m) {
      const float b = weight_value(w_n[(int64_t)m * nk + k], wscale);
      s_w[p * NORB + m] = b;
      lbmax = fmaxf(lbmax, fabsf(b));
      lbmin = fminf(lbmin, b);
    }
  }
  lmin = wave_min(lmin);
  lmax = wave_max(lmax);
  lbmax = wave_max(lbmax);
  lbmin = wave_min(lbmin);
  if ((tid & 63) == 0) {
    s_red[tid >> 6] = lmin;
    s_red[NW + (tid >> 6)] = lmax;
    s_red[2 * NW + (tid >> 6)] = lbmax;
    s_red[3 * NW + (tid >> 6)] = lbmin;
  }
  __syncthreads();
  float emin = s_red[0], emax = s_red[NW], bmax = s_red[2 * NW], bmin = s_red[3 * NW];
  for (int i = 1; i < NW; ++i) {
    emin = fminf(emin, s_red[i]);
    emax = fmaxf(emax, s_red[NW + i]);
    bmax = fmaxf(bmax, s_red[2 * NW + i]);
    bmin = fminf(bmin, s_red[3 * NW + i]);
  }
  emin = uniform(emin);
  emax = uniform(emax);
  bmax = uniform(bmax);
  bmin = uniform(bmin);
  if (!(emin <= emax)) return;  // no finite energy in this tile-band (uniform across the block)
  int J0, J1;
  range_window(emin, emax, a.e0, a.inv_de, a.ne, J0, J1);

  // This lane's cube; corner slot s sits at LDS point pbase + point_offset(s).
  const bool valid = tid < ncubes;
  int pbase = 0;
  if (valid) {
    const int r = tid / tl.cz, cz = tid - r * tl.cz, cx = r / tl.cy, cy = r - cx * tl.cy;
    pbase = cx * PY + cy * PZ + cz;
  }
  auto point_offset = [](int s) { return (s & 1) * PY + ((s >> 1) & 1) * PZ + (s >> 2); };

  // Bound on any bin's sum: sum over tetrahedra with a possibly non-empty window of 12 V bmax / E41.
  float bound = 0.0f, narrow = 0.0f;
  const float c12 = 12.0f * a.V * bmax;
  if (valid) {
#pragma unroll 1
    for (int t = 0; t < 6; ++t) {
      const uint32_t slots = tet_slots(t);
      float lo = __builtin_huge_valf(), hi = -__builtin_huge_valf();
      bool fin = true;
#pragma unroll
      for (int l = 0; l < 4; ++l) {
        const float e = s_eps[pbase + point_offset((slots >> (4 * l)) & 7)];
        fin = fin && __builtin_isfinite(e);
        lo = fminf(lo, e);
        hi = fmaxf(hi, e);
      }
      if (!fin || !(hi > lo)) continue;
      int jlo, jhi;
      energy_window(lo, hi, a.e0, a.inv_de, J0, J1, jlo, jhi);
      if (jlo > jhi + 2) continue;
      const float term = c12 * rcp(hi - lo);
      bound += term;
      if (hi - lo < 2.0f * a.de) narrow += term;
    }
  }
  bound = wave_sum(fminf(bound, 1.0e37f));
  narrow = wave_sum(fminf(narrow, 1.0e37f));
  __syncthreads();  // every lane has read s_red
  if ((tid & 63) == 0) {
    s_red[tid >> 6] = bound;
    s_red[NW + (tid >> 6)] = narrow;
  }
  __syncthreads();
  float B = 0.0f, Bn = 0.0f;
  for (int i = 0; i < NW; ++i) {
    B += s_red[i];
    Bn += s_red[NW + i];
  }
  B = uniform(B);
  Bn = uniform(Bn);
  if (!(B > 0.0f)) return;  // nothing to add (uniform across the block)
  if (MODE == 1) {
    if (tid == 0) {
      int be;
      frexpf(fminf(B, 3.0e38f), &be);
      atomicMax(a.gexp, be);
    }
    return;
  }
  const bool packed = bmin >= 0.0f && Bn <= 0.5f * B;  // uniform across the block
  const int rows = packed ? NPAIR : NORB;
  const int RS = packed ? RSP : RSW;
  // Copies: lane l adds into copy l % CP of a bin (each bin's copies are adjacent words), so the lanes
  // of neighbouring cubes, which usually hit the same bins at the same time, do not serialise on one
  // LDS address. As many copies (up to eight) as keep the tile-band's energy range in one pass.
  const int span = uniform(J1 - J0 + 1);
  const int cpl = span <= (RS >> 3) ? 3 : span <= (RS >> 2) ? 2 : span <= (RS >> 1) ? 1 : 0;  // log2 of the copy count
  const int CP = 1 << cpl;
  const int LC = RS >> cpl;  // bins per pass
  int bexp;
  frexpf(fminf(B, 3.0e38f), &bexp);  // B <= 2^bexp
  const int sexp = uniform(min((packed ? 30 : 62) - bexp, 126));
  const float S = ldexpf(1.0f, sexp);  // B * S <= 2^30 (packed) or 2^62
  // exact mode: shift from this workgroup's fixed point to the common one (negative: to the right)
  const int dshift = MODE == 2 ? exact_scale_exp(*a.gexp, a.lg_units) - sexp : 0;
  // Fold the power-of-two scale into the staged weights (exact): every deposit is then an integer-valued
  // float without a per-orbital multiply.
  for (int q = tid; q < np; q += NT) {
    const int r = small_div(q, by_qz), pz = q - r * qz, px = small_div(r, by_qy), py = r - px * qy;
    float* w = &s_w[(px * PY + py * PZ + pz) * NORB];
#pragma unroll
    for (int m = 0; m < NORB; ++m) w[m] *= S;
  }
  __syncthreads();

  for (int c0 = J0; c0 <= J1; c0 += LC) {
    const int c1 = min(c0 + LC - 1, J1);
    const int L = c1 - c0 + 1;
    const int LW = L << cpl;  // words per row in this pass
    // The lane index again, opaque: the addresses derived from it are formed in each pass instead of
    // being kept live (in scratch) over the whole unit.
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    for (int q = tid; q < rows * LW; q += NT) {
      const int r = q / LW;
      s_hist[r * RS + (q - r * LW)] = 0ull;
    }
    __syncthreads();
    if (valid) {
#pragma unroll 1
      for (int t = 0; t < 6; ++t) {
        const uint32_t slots = tet_slots(t);
        float e[4];
        int pt[4];  // LDS point of each corner, carried through the sort
#pragma unroll
        for (int l = 0; l < 4; ++l) {
          pt[l] = pbase + point_offset((slots >> (4 * l)) & 7);
          e[l] = s_eps[pt[l]];
        }
        if (!finite4(e[0], e[1], e[2], e[3])) continue;
        sort4(e, pt);
        int jlo, jhi;
        energy_window(e[0], e[3], a.e0, a.inv_de, c0, c1, jlo, jhi);
        if (jlo > jhi + 2) continue;  // empty even after moving both ends by one
        const TetSetup cs = tet_setup(e, a.e0, a.V);
        tet_window(cs, a.de, c0, c1, jlo, jhi);
        if (jlo > jhi) continue;
        float bb[4][NORB];
#pragma unroll
        for (int l = 0; l < 4; ++l) {
#pragma unroll
          for (int m = 0; m < NORB; ++m) bb[l][m] = s_w[pt[l] * NORB + m];
        }
        // The window splits into the three energy cases at jA and jB.
        int jA, jB;
        case_split(cs, a.de, a.inv_de, jlo, jhi, jA, jB);
        // Packed: two orbitals per 64-bit word as unsigned 32-bit fields; every term is non-negative
        // (the weights are, and the corner weights are clamped at zero against rounding), so the
        // truncating conversion of 0.5 + v rounds v to the nearest integer (halves up).
        auto deposit = [&](int j, const float g[4]) {
          unsigned long long* h = &s_hist[((j - c0) << cpl) + (tid & (CP - 1))];
          if (packed) {
#pragma unroll
            for (int pr = 0; pr < NPAIR; ++pr) {
              const int m0 = 2 * pr, m1 = 2 * pr + 1;
              float v0 = __builtin_fmaf(g[0], bb[0][m0], 0.5f);
              v0 = __builtin_fmaf(g[1], bb[1][m0], v0);
              v0 = __builtin_fmaf(g[2], bb[2][m0], v0);
              v0 = __builtin_fmaf(g[3], bb[3][m0], v0);
              unsigned long long word = (unsigned long long)(unsigned)v0;
              if (m1 < NORB) {
                float v1 = __builtin_fmaf(g[0], bb[0][m1], 0.5f);
                v1 = __builtin_fmaf(g[1], bb[1][m1], v1);
                v1 = __builtin_fmaf(g[2], bb[2][m1], v1);
                v1 = __builtin_fmaf(g[3], bb[3][m1], v1);
                word |= (unsigned long long)(unsigned)v1 << 32;
              }
              atomicAdd(&h[pr * RSP], word);
            }
          } else {
#pragma unroll
            for (int m = 0; m < NORB; ++m) {
              const float v = g[0] * bb[0][m] + g[1] * bb[1][m] + g[2] * bb[2][m] + g[3] * bb[3][m];
              atomicAdd(&h[m * RSW], (unsigned long long)__float2ll_rn(v));
            }
          }
        };
        // One loop over the whole window: a wavefront runs as long as its longest window instead of
        // the sum of its longest per-case ranges; each energy evaluates its own case's weights.
        float coef[4][4];
        if (jB > jA) corner_dos_B_coeffs(cs, a.V, coef);
        for (int j = jlo; j <= jhi; ++j) {
          float g[4];
          if (j <= jA) {
            corner_dos_A(cs, local_x(cs, j, a.de), g);
            g[0] = fmaxf(g[0], 0.0f);  // g[1..3] are products of non-negative factors
          } else if (j <= jB) {
            corner_dos_B_poly(coef, local_z(cs, j, a.de), g);
#pragma unroll
            for (int l = 0; l < 4; ++l) g[l] = fmaxf(g[l], 0.0f);
          } else {
            corner_dos_C(cs, local_y(cs, j, a.de), g);
            g[3] = fmaxf(g[3], 0.0f);
          }
          deposit(j, g);
        }
      }
    }
    __syncthreads();
    for (int q = tid; q < L * NORB; q += NT) {
      const int r = q / NORB, m = q - r * NORB;
      const int row = packed ? (m >> 1) : m;
      const unsigned long long* hw = &s_hist[row * RS + (r << cpl)];
      if constexpr (MODE == 2) {
        // exact sum of the copies in this workgroup's fixed point (|v| <= B S <= 2^62), then one
        // rounding (halves up) to the common fixed point
        long long v = 0;
        for (int c = 0; c < CP; ++c) {
          const unsigned long long w = hw[c];
          v += packed ? (long long)(unsigned)((m & 1) ? (w >> 32) : (w & 0xffffffffull)) : (long long)w;
        }
        long long q;
        if (dshift >= 0) q = (long long)((unsigned long long)v << dshift);
        else if (dshift > -63) q = (v + (1ll << (-dshift - 1))) >> (-dshift);
        else q = 0;  // |v| < 2^62 <= half a unit of the common fixed point
        if (q != 0) atomicAdd(&a.gacc[(int64_t)(c0 + r) * NORB + m], (unsigned long long)q);
      } else {
        double sum = 0.0;
        for (int c = 0; c < CP; ++c) {
          const unsigned long long w = hw[c];
          sum += packed ? (double)(unsigned)((m & 1) ? (w >> 32) : (w & 0xffffffffull)) : (double)(long long)w;
        }
        // the scale formed here rather than kept live over the passes (a register less there)
        if (sum != 0.0) atomic_add_global(&a.dos[(int64_t)(c0 + r) * NORB + m], (float)ldexp(sum, -sexp));
      }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------------------------
// Spline form (tetra_spline.h): one lane per grid point of the tile instead of one per cube.

template <int NORB>
struct SplineFixed {
  double u[kKnotPad];  // knots: energies in grid steps
  float f[NP];         // the energies, for the search for degenerate tetrahedra; infinite where not finite
  float wlo[kWeightPad];
  float w[NP * NORB];
  float whi[kWeightPad];
  uint32_t skip[NP];
  unsigned short queue[kQueue];
  float red[3 * NWMAX];
  double dred[NWMAX];
  int nq;
};
template <int NORB>
constexpr int spline_words() { return (kLdsBytes - 64 - (int)sizeof(SplineFixed<NORB>)) / 8; }
template <int NORB>
struct SplineShared : SplineFixed<NORB> {
  double hist[spline_words<NORB>()];
};

template <int NORB>
union FwdShared {
  GeneralShared<NORB> general;
  SplineShared<NORB> spline;
};

// The unit by the spline form; false (uniform across the workgroup) when the tile-band is not for it.
// MODE 0: FP64 sums, flushed with float atomics. MODE 2: 64-bit integers, so that nothing depends on the
// order of the atomics: a first sweep over the points finds the largest entry, which fixes the scale.
// MODE 3: the increments N(E_j) - N(E_{j-1}) of the number of states on the grid e0 + (j + joff) de
// (everything below the grid at index 0) instead of the DOS: fifth differences of quartics, and the same
// four running sums.
template <int NORB, typename WT, int MODE>
__device__ __forceinline__ bool spline_unit(const FwdArgs& a, int unit, SplineShared<NORB>& sh) {
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
  const double e0 = a.e0, inv_de = a.inv_ded, joff = INC ? a.joff : 0.0;
  if (nk >= (1ll << 29)) return false;  // byte offsets within a plane are 32-bit below
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
      ahead_e[i] = load_at(eps_n, k);
#pragma unroll
      for (int m = 0; m < NORB; ++m) ahead_w[i][m] = load_at(w_n + (int64_t)m * nk, k);
    }
  }
  for_lanes(kKnotPad, [&](int i) { sh.u[i] = kFarKnot; });
  for_lanes(kWeightPad, [&](int i) { sh.wlo[i] = sh.whi[i] = 0.0f; });
  for_lanes(NP, [&](int i) { sh.skip[i] = 0u; });
  if (np < NP)  // every word a neighbour offset can reach holds a finite value
    for_lanes(NP * NORB, [&](int i) { sh.w[i] = 0.0f; });
  if (tid == 0) sh.nq = 0;
  __syncthreads();
  float lmin = __builtin_huge_valf(), lmax = -__builtin_huge_valf(), lbmax = 0.0f, lsum = 0.0f;
  auto stage = [&](int q, float e, auto&& weight) {
    int px, py, pz;
    split(q, px, py, pz);
    const int p = px * PY + py * PZ + pz;
    const bool finite = __builtin_isfinite(e);
    sh.f[p] = finite ? e : __builtin_huge_valf();
    if (finite) {
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
      stage(q, load_at(eps_n, k), [&](int m) { return load_at(w_n + (int64_t)m * nk, k); });
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
  if (!(emin <= emax)) return true;  // no finite energy
  const double umin = ((double)emin - e0) * inv_de - joff, umax = ((double)emax - e0) * inv_de - joff;
  auto index = [&](float e, bool above, double lo, double top) {  // INC
    return energy_index(e, e0, (double)a.de, inv_de, joff, above, lo, top);
  };
  // above the energy grid (a flat tetrahedron on its last energy has all its states there)
  if (INC ? index(emin, false, -1.0, (double)a.ne) > (double)(a.ne - 1) : !(umin < (double)(a.ne - 1))) return true;
  if (!(uniform(bmax) < 3.0e38f)) return false;
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
            sum += top < __builtin_huge_valf() ? (double)b : 0.0;
          }
        });
        if (sum != 0.0) unsafeAtomicAdd(&sh.hist[m], sum);
      }
      __syncthreads();
      for_lanes(NORB, [&](int m) { atomic_add_global(&a.dos[m], (float)(sh.hist[m] * a.Vd)); });
    }
    return true;
  }
  // Rows of the sums: from the first grid energy at or above the lowest knot (below the grid's first
  // energy too) to the last one below the highest (the first at or above it for the increments).
  const double rows_d = INC ? fmin(fmax(ceil(umax), index(emax, false, -1.0, (double)a.ne)), (double)(a.ne - 1)) + 1.0 - floor(umin)
                            : fmin(ceil(umax), (double)a.ne) - floor(umin);
  if (!(rows_d + NE + 2 <= (double)spline_words<NORB>())) return false;
  const int base = uniform((int)floor(umin)), rows = uniform((int)rows_d);
  const float J = (float)rows, limit = (MODE == 2 ? kDegenerateExact : a.degenerate) * J * J * J;

  // Degenerate tetrahedra: their bits at their corner points, and a queue of those with finite corners.
  const int by_cz = small_inverse(cz), by_cy = small_inverse(cy);
  for_lanes(ncubes, [&](int c) {
    const int r = small_div(c, by_cz), iz = c - r * cz, ix = small_div(r, by_cy), iy = r - ix * cy;
    const float* fc = &sh.f[ix * PY + iy * PZ + iz];
    float f[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) f[s] = fc[(s & 1) * PY + ((s >> 1) & 1) * PZ + (s >> 2)];
    uint32_t finite;
    const uint32_t out = left_out(f, limit, finite, a.inv_de);
    if (out) {
#pragma unroll
      for (int t = 0; t < 6; ++t) {
        if (!((out >> t) & 1u)) continue;
        if ((finite >> t) & 1u) {
          const int at = atomicAdd(&sh.nq, 1);
          if (at < kQueue) sh.queue[at] = (unsigned short)(c * 6 + t);
        }
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
  const int nq = uniform(sh.nq);
  if (nq > kQueue) return false;

  // As many orbitals at a time as the histogram holds, then as many copies of it (a lane adds into copy
  // lane mod copies: neighbouring points often share a bin).
  const int RS = (rows + NE + 1) | 1;
  int group = NORB;
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
    if (!(ju - base < (double)rows)) return;  // above the last row (or not finite)
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
    const int row = (int)(ju - base);
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

  // Degenerate tetrahedra, energy by energy, 16 lanes each: the fourth differences 1, -4, 6, -4, 1 of the
  // value at one energy. Called by the lanes in reverse order next to the points, of which the last waves
  // have fewer.
  auto degenerate = [&](int i16, int m0, int m1, double unit, auto&& add) {
    const int i = i16 >> 4;
    const int item = sh.queue[i], c = item / 6, t = item - 6 * c;
    const int r = small_div(c, by_cz), iz = c - r * cz, ix = small_div(r, by_cy), iy = r - ix * cy;
    const uint32_t slots = tet_slots(t);
    float e[4];
    int pt[4];
#pragma unroll
    for (int l = 0; l < 4; ++l) {
      const int s = (slots >> (4 * l)) & 7;
      const int px = ix + (s & 1), py = iy + ((s >> 1) & 1), pz = iz + (s >> 2);
      e[l] = eps_n[((int64_t)wrap(x0 + px, a.n1) * a.n2 + wrap(y0 + py, a.n2)) * a.n3 + wrap(z0 + pz, a.n3)];
      pt[l] = px * PY + py * PZ + pz;
    }
    sort4(e, pt);
    if (!INC && !(e[3] > e[0])) return;
    auto put = [&](int j, double g0, double g1, double g2, double g3) {
#pragma unroll 1
      for (int m = m0; m < m1; ++m) {
        const float* w = sh.w + m * NP;
        const double v = unit * (g0 * w[pt[0]] + g1 * w[pt[1]] + g2 * w[pt[2]] + g3 * w[pt[3]]);
        Acc* h = &hist[(m - m0) * RS + j - base];
        add(h, v, 1);
        add(h + 1, v, -4);
        add(h + 2, v, 6);
        add(h + 3, v, -4);
        add(h + 4, v, 1);
      }
    };
    if constexpr (INC) {
      const NosVolumes c = nos_volumes(e);
      const int full = (int)index(e[3], false, base, (double)a.ne), js = min(full, base + rows - 1);
      const int ja = min((int)index(e[0], true, base, (double)a.ne), js);
      for (int j = ja + (i16 & 15); j <= js; j += 16) {
        double w0[4] = {0.0, 0.0, 0.0, 0.0}, w1[4] = {1.0, 1.0, 1.0, 1.0};
        if (j > ja) corner_nos(c, 1.0, e0 + (j - 1 + joff) * (double)a.de, w0);
        if (j < full) corner_nos(c, 1.0, e0 + (j + joff) * (double)a.de, w1);
        put(j, w1[0] - w0[0], w1[1] - w0[1], w1[2] - w0[2], w1[3] - w0[3]);
      }
    } else {
      tet_energies(e, a, 0, a.ne - 1, i16 & 15, 16, [&](int j, const float g[4]) { put(j, g[0], g[1], g[2], g[3]); });
    }
  };

  for (int m0 = 0; m0 < NORB; m0 += group) {
    const int m1 = min(m0 + group, NORB), gm = m1 - m0;
    for_lanes(copies * plane, [&](int i) { hist[i] = Acc(0); });
    int sexp = 0;
    if constexpr (MODE == 2) {
      // Fixed point: entries below 2^51, sums of every bin (below 2^gexp) below 2^62.
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
      sexp = min(51 - dexp, 62 - *a.gexp);
    }
    __syncthreads();
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
    for_lanes(16 * nq, [&](int i16) {
      degenerate(i16, m0, m1, MODE == 2 ? ldexp(1.0, sexp) : INC ? a.Vd : 1.0, [&](Acc* h, double v, int times) {
        if constexpr (MODE == 2)
          atomicAdd(reinterpret_cast<unsigned long long*>(h), (unsigned long long)(times * (long long)rint(v)));
        else
          unsafeAtomicAdd(h, v * times);
      });
    }, true);
    __syncthreads();
    running_sums(hist, gm, RS, plane, copies, rows);
    __syncthreads();
    const int lo = max(-base, 0);
    if (INC && lo > 0 && a.shift == 0) {  // increments below the grid count at its first energy
      for_lanes(lo * gm, [&](int i) {
        const int m = i / lo;
        unsafeAtomicAdd(&sh.hist[m * RS + lo], sh.hist[m * RS + i - m * lo]);
      });
      __syncthreads();
    }
    for_lanes((rows - lo) * gm, [&](int i) {
      const int q = gm == NORB ? i / NORB : i / gm, r = lo + q, m = i - q * gm;
      const Acc v = hist[m * RS + r];
      const int64_t at = (int64_t)(base + r) * NORB + m0 + m;
      if constexpr (MODE == 2) {
        const int dshift = exact_scale_exp(*a.gexp, a.lg_units) - sexp;
        long long fixed;
        if (dshift >= 0) fixed = (long long)((unsigned long long)v << dshift);
        else if (dshift > -63) fixed = (v + (1ll << (-dshift - 1))) >> (-dshift);
        else fixed = 0;
        if (fixed != 0) atomicAdd(&a.gacc[at], (unsigned long long)fixed);
      } else if constexpr (INC) {
        if (v != 0.0 && base + r >= a.shift)
          atomic_add_global(&a.dos[at - a.shift * NORB], (float)(v * a.out_scale));
      } else {
        if (v != 0.0) atomic_add_global(&a.dos[at], (float)v);
      }
    });
    __syncthreads();
  }

  return true;
}

// One work unit: the spline form, or the general one for the tile-bands that are not for it.
template <int NORB, typename WT, int MODE>
__device__ __forceinline__ void forward_unit(const FwdArgs& a, int unit, FwdShared<NORB>& sh) {
  if (spline_unit<NORB, WT, MODE>(a, unit, sh.spline)) return;
  __syncthreads();
  general_unit<NORB, WT, MODE>(a, unit, sh.general);
}

template <int NORB, typename WT, int MODE>
__global__ __launch_bounds__(NTMAX, kWaves) void dos_forward_kernel(FwdArgs a) {
  // XCD-aware mapping: hardware dispatches block b to XCD b % 8; give each XCD a contiguous range.
  const int b = blockIdx.x;
  const int unit = (b % NXCD) * a.per_xcd + b / NXCD;
  if (unit >= a.nunits) return;
  if constexpr (MODE == 1) {
    __shared__ GeneralShared<NORB> sh;
    general_unit<NORB, WT, 1>(a, unit, sh);
  } else {
    __shared__ FwdShared<NORB> sh;
    forward_unit<NORB, WT, MODE>(a, unit, sh);
  }
}

// ---------------------------------------------------------------------------------------------
// Batched forward: one launch over the flattened (item, band, tile) units of up to kMaxBatch problems with
// the same orbital count, a workgroup per unit.

template <int NORB, typename WT>
__global__ __launch_bounds__(NTMAX, kWaves) void dos_batched_kernel(BatchArgs b) {
  __shared__ FwdShared<NORB> sh;
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
  a.degenerate = it.degenerate;
  forward_unit<NORB, WT, 0>(a, u - it.unit_begin, sh);
}

// Zero every item's DOS (blockIdx.y = item).
__global__ void batched_zero_kernel(BatchArgs b, int norb) {
  const BatchItem& it = b.it[blockIdx.y];
  const int64_t n = (int64_t)it.ne * norb;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    it.dos[i] = 0.0f;
}

template <int NORB, int MODE>
hipError_t launch_fwd_mode(const FwdArgs& a, int grid, hipStream_t s) {
  if (a.wtype == TETRA_W_F16)
    hipLaunchKernelGGL((dos_forward_kernel<NORB, _Float16, MODE>), dim3(grid), dim3(a.lanes), 0, s, a);
  else if (a.wtype == TETRA_W_C32)
    hipLaunchKernelGGL((dos_forward_kernel<NORB, float2, MODE>), dim3(grid), dim3(a.lanes), 0, s, a);
  else
    hipLaunchKernelGGL((dos_forward_kernel<NORB, float, MODE>), dim3(grid), dim3(a.lanes), 0, s, a);
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
