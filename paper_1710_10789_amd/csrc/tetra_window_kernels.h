// Forward pass over every tetrahedron's window of energies (gfx950), for calls with so few energies that the spline form
// (tetra_forward_kernels.h), whose work does not depend on their number, is the slower one; which those are: few_energies
// in tetra_forward.hip.
//
// One workgroup of 256 lanes per (tile of TX x TY x TZ cubes, band): the tile's grid points are staged once in LDS,
// a lane per cube goes over its six tetrahedra (Table I), sorts the corner energies and adds the contribution at every
// energy inside (E1, E4) to an LDS histogram of 64-bit fixed-point integers. Every contribution is non-negative (a corner
// weight is the section integral of a barycentric coordinate) and a tetrahedron's point DOS never exceeds
// 3 V_T/(V_G E41), so with bmax = max |b| of the tile the bound B = sum 12 V bmax / E41 over the tetrahedra with a
// non-empty window fixes a power-of-two scale S with B*S <= 2^62 (two's complement, so signed weights work too). With
// non-negative weights and a bound that narrow tetrahedra (E41 < 2 de) do not dominate, two orbitals share one 64-bit
// atomic as two 32-bit fields with B*S <= 2^30 (no carry between fields). One global float atomic per touched bin.
// Bound by vector instruction issue, about 90 per energy of a window. 64^3 x 8 x 8 x 32 0.152 ms against 0.163 ms in the
// spline form, in the exact mode 0.258 against 0.339 ms. Weights aligned to 16 bytes (a point's in two loads; without, the
// same kernel takes 0.205 ms), 5 waves per SIMD with 7 and 8 orbitals (6 would spill).
#pragma once

#include "tetra_device.h"
#include "tetra_spline_tile.h"
#include "tetra_weights.h"

namespace tetra {

namespace {

// Common fixed point of the exact mode: with E the largest bound exponent of any workgroup (each
// workgroup's bins sum to at most 2^E in magnitude) and L = ceil(log2(workgroups)), the total of any
// bin is below 2^(E + L), so the scale 2^(62 - E - L) keeps every partial and total sum of the
// 64-bit two's-complement accumulator in range.
__device__ __forceinline__ int exact_scale_exp(int gexp, int lg_units) { return 62 - gexp - lg_units; }

// Histogram words and the waves per SIMD the kernels are held to.
template <int NORB>
constexpr int window_words() { return NORB <= 8 ? 1280 : NORB == 16 ? 1344 : 2048; }
template <int NORB>
constexpr int window_waves() { return NORB <= 6 ? 6 : NORB <= 8 ? 5 : NORB == 16 ? 4 : 1; }

template <int NORB>
struct WindowShared {
  alignas(16) float w[kTilePointsMax * NORB];  // read a point's weights at a time
  float eps[kTilePointsMax];
  unsigned long long hist[window_words<NORB>()];
  float red[4 * (kTileCubes / 64)];
};

// One work unit; every lane of the workgroup calls it.
// MODE 0: DOS with per-workgroup scales, flushed with float atomics;
// 1: only the workgroup's bound exponent, into *gexp (atomicMax: independent of the order);
// 2: DOS with per-workgroup scales as in mode 0; each bin's exact per-workgroup sum is rounded once
//    to the common fixed point fixed by *gexp and added to gacc with a 64-bit integer atomic. Both
//    steps are independent of the order in which workgroups run, so the result is bitwise
//    reproducible.
template <int NORB, typename WT, int MODE>
__device__ __forceinline__ void window_unit(const FwdArgs& a, int unit, WindowShared<NORB>& sh) {
  constexpr int NT = kTileCubes, NW = NT >> 6;
  constexpr int NPAIR = (NORB + 1) / 2;
  // Histogram rows (one per orbital pair in the packed form, one per orbital in the wide form) have a
  // fixed, odd stride in 64-bit words: the row offsets of a deposit are immediates, and the flush
  // reads across rows without bank conflicts.
  constexpr int HCAP = window_words<NORB>();
  constexpr int RSP = (HCAP / NPAIR - 1) | 1, RSW = (HCAP / NORB - 1) | 1;
  float* const s_eps = sh.eps;
  float* const s_w = sh.w;
  unsigned long long* const s_hist = sh.hist;
  float* const s_red = sh.red;

  const int TX = a.s1, TY = a.s2, TZ = a.s3;
  const int PY = TY + 1, PZ = TZ + 1;
  const int NP = (TX + 1) * PY * PZ;
  const int band = unit / a.ntiles;
  const int tile = unit - band * a.ntiles;
  const int tz = tile % a.t3;
  const int ty = (tile / a.t3) % a.t2;
  const int tx = tile / (a.t3 * a.t2);
  const int x0 = tx * TX, y0 = ty * TY, z0 = tz * TZ;
  const int tid = threadIdx.x;
  const int64_t nk = (int64_t)a.n1 * a.n2 * a.n3;
  const float* eps_n = a.eps + (int64_t)band * nk;
  const WT* w_n = static_cast<const WT*>(a.w) + (int64_t)band * NORB * nk;
  const float wscale = a.w_scale ? a.w_scale[band] : 1.0f;

  // Stage the tile's grid points (periodic wrap) and find their energy range.
  float lmin = __builtin_huge_valf(), lmax = -__builtin_huge_valf(), lbmax = 0.0f, lbmin = 0.0f;
  for (int p = tid; p < NP; p += NT) {
    const int pz = p % PZ, py = (p / PZ) % PY, px = p / (PZ * PY);
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
#pragma unroll
  for (int i = 1; i < NW; ++i) {
    emin = fminf(emin, s_red[i]);
    emax = fmaxf(emax, s_red[NW + i]);
    bmax = fmaxf(bmax, s_red[2 * NW + i]);
    bmin = fminf(bmin, s_red[3 * NW + i]);
  }
  if (!(emin <= emax)) return;  // no finite energy in this tile-band (uniform across the block)
  int J0, J1;
  range_window(emin, emax, a.e0, a.inv_de, a.ne, J0, J1);

  // This lane's cube; corner slot s sits at LDS point pbase + point_offset(s).
  const int cz = tid % TZ, cy = (tid / TZ) % TY, cx = tid / (TZ * TY);
  const bool valid = (x0 + cx < a.n1) && (y0 + cy < a.n2) && (z0 + cz < a.n3);
  const int pbase = (cx * PY + cy) * PZ + cz;
  auto point_offset = [PY, PZ](int s) { return (s & 1) * (PY * PZ) + ((s >> 1) & 1) * PZ + (s >> 2); };

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
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    B += s_red[i];
    Bn += s_red[NW + i];
  }
  if (!(B > 0.0f)) return;  // nothing to add (uniform across the block)
  if constexpr (MODE == 1) {
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
  const int span = J1 - J0 + 1;
  const int cpl = span <= (RS >> 3) ? 3 : span <= (RS >> 2) ? 2 : span <= (RS >> 1) ? 1 : 0;  // log2 of the copy count
  const int CP = 1 << cpl;
  const int LC = RS >> cpl;  // bins per pass
  int bexp;
  frexpf(fminf(B, 3.0e38f), &bexp);  // B <= 2^bexp
  const int sexp = min((packed ? 30 : 62) - bexp, 126);
  const float S = ldexpf(1.0f, sexp);  // B * S <= 2^30 (packed) or 2^62
  // exact mode: shift from this workgroup's fixed point to the common one (negative: to the right)
  const int dshift = MODE == 2 ? exact_scale_exp(*a.gexp, a.lg_units) - sexp : 0;
  // Fold the power-of-two scale into the staged weights (exact): every deposit is then an integer-valued
  // float without a per-orbital multiply.
  for (int q = tid; q < NP * NORB; q += NT) s_w[q] *= S;
  __syncthreads();

  for (int c0 = J0; c0 <= J1; c0 += LC) {
    const int c1 = min(c0 + LC - 1, J1);
    const int L = c1 - c0 + 1;
    const int LW = L << cpl;  // words per row in this pass
    // The lane index again, opaque: the addresses derived from it are formed in each pass instead of
    // being kept live (in scratch) over the whole unit. (Not in the exact mode's second pass, whose
    // register allocation it upsets.)
    int tid = threadIdx.x;
    if constexpr (MODE != 2) asm volatile("" : "+v"(tid));
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

template <int NORB, typename WT, int MODE>
__global__ __launch_bounds__(kTileCubes, window_waves<NORB>()) void dos_window_kernel(FwdArgs a) {
  __shared__ WindowShared<NORB> sh;
  const int b = blockIdx.x;
  const int unit = (b % NXCD) * a.per_xcd + b / NXCD;  // each XCD a contiguous range of units
  if (unit < a.nunits) window_unit<NORB, WT, MODE>(a, unit, sh);
}

}  // namespace

}  // namespace tetra
