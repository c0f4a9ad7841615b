// Number-of-states kernel: orbital-resolved number of states and bin-averaged DOS on gfx950.
//
// N[j][m] = sum over the tetrahedra of Table I, bands n and corners l of b[n][m][k_l] w_{n,l}(E_j):
// eq. (BZintegral) with X = b of eq. (matrixelements) and the step occupation at E_j, summed by the
// tetrahedron method (eqs. tetmethod, tetracontrib) with the integrated corner weights w_l of the five
// energy cases of Sec. II.C (arXiv:1710.10789).
//
// A tetrahedron-band's w_l(E) is zero up to E1, a polynomial on (E1, E4) and V_T/(4 V_G) from E4 on,
// so over the grid it is described by its increments w_l(E_j) - w_l(E_{j-1}), non-zero only from the
// first E_j > E1 to the first E_j >= E4. The kernel adds those increments (contracted with the corner
// weights b) into a histogram, and a scan over j afterwards sums them to N: the work follows the
// tetrahedron's window, not the energies above it. The increments on the grid of midpoints
// E_j -+ de/2, divided by de, are the bin averages (N(E_j + de/2) - N(E_j - de/2)) / de of the DOS,
// whose sum over the bins telescopes to the difference of N at the two outer edges.
//
// Work decomposition and accumulation as in the forward kernels, whose spline form (tetra_forward_kernels.h,
// MODE 3) does nearly all of it: a grid point adds the five fifth differences of its quartic per orbital, and
// four running sums give the tile's increments. The loop over every tetrahedron's energies that it replaces
// took 0.45 ms for 64^3 x 8 x 8 x 1000 and, in FP64 where a tetrahedron spanned more than 64 energies,
// 1.23 ms for 24^3 x 8 x 8 x 4096.
// Tile-bands that the spline form is not for take general_nos: one lane per cube, the increments of every
// tetrahedron energy by energy (volumes in FP64: an increment is a small difference of values up to V),
// added to an FP64 histogram in LDS.
#pragma once

#include "tetra_forward_kernels.h"

namespace tetra {

namespace {

constexpr int kNosWords = 3584;  // histogram words
template <int NORB>
struct NosGeneral {
  float eps[NP];
  float w[NP * NORB];
  float red[2 * NWMAX];
  double hist[kNosWords];
};
template <int NORB>
union NosShared {
  NosGeneral<NORB> general;
  SplineShared<NORB> spline;
};

template <int NORB, typename WT>
__device__ __forceinline__ void general_nos(const FwdArgs& a, int unit, NosGeneral<NORB>& sh) {
  static_assert(sizeof(NosGeneral<NORB>) <= kLdsBytes, "LDS");
  constexpr int RS = (kNosWords / NORB - 1) | 1;  // energies per pass
  int band;
  const Tile tl = unit_tile(a, unit, band);
  const int cy = tl.cy, cz = tl.cz, qy = cy + 1, qz = cz + 1, np = (tl.cx + 1) * qy * qz, ncubes = tl.cx * cy * cz;
  const int tid = threadIdx.x, NW = blockDim.x >> 6;
  const int64_t nk = (int64_t)a.n1 * a.n2 * a.n3;
  const float* eps_n = a.eps + (int64_t)band * nk;
  const WT* w_n = static_cast<const WT*>(a.w) + (int64_t)band * NORB * nk;
  const float wscale = a.w_scale ? a.w_scale[band] : 1.0f;
  float lmin = __builtin_huge_valf(), lmax = -__builtin_huge_valf();
  for_lanes(np, [&](int q) {
    const int r = q / qz, pz = q - r * qz, px = r / qy, py = r - px * qy, p = px * PY + py * PZ + pz;
    const int64_t k = ((int64_t)wrap(tl.x0 + px, a.n1) * a.n2 + wrap(tl.y0 + py, a.n2)) * a.n3 + wrap(tl.z0 + pz, a.n3);
    const float e = eps_n[k];
    sh.eps[p] = e;
    if (__builtin_isfinite(e)) {
      lmin = fminf(lmin, e);
      lmax = fmaxf(lmax, e);
    }
#pragma unroll 1
    for (int m = 0; m < NORB; ++m) sh.w[m * NP + p] = weight_value(w_n[(int64_t)m * nk + k], wscale);
  });
  lmin = wave_min(lmin);
  lmax = wave_max(lmax);
  if ((tid & 63) == 0) {
    sh.red[tid >> 6] = lmin;
    sh.red[NW + (tid >> 6)] = lmax;
  }
  __syncthreads();
  float emin = sh.red[0], emax = sh.red[NW];
  for (int i = 1; i < NW; ++i) {
    emin = fminf(emin, sh.red[i]);
    emax = fmaxf(emax, sh.red[NW + i]);
  }
  emin = uniform(emin);
  emax = uniform(emax);
  if (!(emin <= emax)) return;  // no finite energy
  const double e0 = a.e0, de = a.de, inv_de = a.inv_ded, joff = a.joff, top = (double)(a.ne - 1);
  // grid index of the first energy above (shift 1) or at or above (shift 0) an energy, kept inside the grid
  auto index = [&](float e, bool above) { return (int)energy_index(e, e0, de, inv_de, joff, above, 0.0, top + 1.0); };
  const int J0 = uniform(index(emin, false)), J1 = min(uniform(index(emax, false)), a.ne - 1);
  for (int c0 = J0; c0 <= J1; c0 += RS) {
    const int c1 = min(c0 + RS - 1, J1), L = c1 - c0 + 1;
    for_lanes(NORB * RS, [&](int i) { sh.hist[i] = 0.0; });
    __syncthreads();
    for_lanes(ncubes, [&](int c) {
      const int r = c / cz, iz = c - r * cz, ix = r / cy, iy = r - ix * cy, p = ix * PY + iy * PZ + iz;
#pragma unroll 1
      for (int t = 0; t < 6; ++t) {
        const uint32_t slots = tet_slots(t);
        float e[4];
        int pt[4];
#pragma unroll
        for (int l = 0; l < 4; ++l) {
          const int s = (slots >> (4 * l)) & 7;
          pt[l] = p + (s & 1) * PY + ((s >> 1) & 1) * PZ + (s >> 2);
          e[l] = sh.eps[pt[l]];
        }
        if (!finite4(e[0], e[1], e[2], e[3])) continue;
        sort4(e, pt);
        const int js = index(e[3], false), ja = min(index(e[0], true), js);  // increments at [ja, js]
        const int j1 = min(js, c1);
        if (ja > c1 || j1 < c0) continue;
        const NosVolumes v = nos_volumes(e);
        const int j0 = max(ja, c0);
        double prev[4] = {0.0, 0.0, 0.0, 0.0};  // nothing below the first increment, everything from the last one on
        if (j0 > ja) corner_nos(v, a.Vd, e0 + (j0 - 1 + joff) * de, prev);
        for (int j = j0; j <= j1; ++j) {
          double cur[4] = {a.Vd, a.Vd, a.Vd, a.Vd};
          if (j < js) corner_nos(v, a.Vd, e0 + (j + joff) * de, cur);
          const double g0 = cur[0] - prev[0], g1 = cur[1] - prev[1], g2 = cur[2] - prev[2], g3 = cur[3] - prev[3];
#pragma unroll 1
          for (int m = 0; m < NORB; ++m) {
            const float* w = sh.w + m * NP;
            const double v = g0 * w[pt[0]] + g1 * w[pt[1]] + g2 * w[pt[2]] + g3 * w[pt[3]];
            if (v == v) unsafeAtomicAdd(&sh.hist[m * RS + j - c0], v);  // a weight that is no number adds nothing
          }
#pragma unroll
          for (int l = 0; l < 4; ++l) prev[l] = cur[l];
        }
      }
    });
    __syncthreads();
    for_lanes(L * NORB, [&](int i) {
      const int r = i / NORB, m = i - r * NORB;
      const double v = sh.hist[m * RS + r];
      const int row = c0 + r - a.shift;
      if (v != 0.0 && row >= 0) atomic_add_global(&a.dos[(int64_t)row * NORB + m], (float)(v * a.out_scale));
    });
    __syncthreads();
  }
}

template <int NORB, typename WT>
__global__ __launch_bounds__(NTMAX, kWaves) void nos_kernel(FwdArgs a) {
  __shared__ NosShared<NORB> sh;
  const int b = blockIdx.x;
  const int unit = (b % NXCD) * a.per_xcd + b / NXCD;  // XCD-aware: contiguous tiles per XCD
  if (unit >= a.nunits) return;
  if (spline_unit<NORB, WT, 3>(a, unit, sh.spline)) return;
  __syncthreads();
  general_nos<NORB, WT>(a, unit, sh.general);
}

}  // namespace

template <int NORB>
hipError_t launch_nos(const FwdArgs& a, int grid, hipStream_t s) {
  if (a.wtype == TETRA_W_F16)
    hipLaunchKernelGGL((nos_kernel<NORB, _Float16>), dim3(grid), dim3(a.lanes), 0, s, a);
  else if (a.wtype == TETRA_W_C32)
    hipLaunchKernelGGL((nos_kernel<NORB, float2>), dim3(grid), dim3(a.lanes), 0, s, a);
  else
    hipLaunchKernelGGL((nos_kernel<NORB, float>), dim3(grid), dim3(a.lanes), 0, s, a);
  return hipGetLastError();
}

}  // namespace tetra
