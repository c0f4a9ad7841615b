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
// Work decomposition and accumulation as in the forward kernels (tetra_forward_kernels.h, MODE 3): a grid point adds
// the five fifth differences of its quartic per orbital, and four running sums give the tile's increments. The loop
// over every tetrahedron's energies that it replaces took 0.45 ms for 64^3 x 8 x 8 x 1000 and, in FP64 where a
// tetrahedron spanned more than 64 energies, 1.03 ms for 24^3 x 8 x 8 x 4096; now 0.197 and 0.040 ms.
// Tetrahedra with nearly equal corner energies are summed energy by energy: volumes in FP64 (an increment is a small
// difference of values up to V), their differences with the weights in FP32. Layered bands, 64^3 x 4 x 8 x 1000:
// 0.61 ms with the loop, 0.81 ms (3.2 ms with FP64 products into one plane of the histogram).
#pragma once

#include "tetra_forward_kernels.h"

namespace tetra {

namespace {

template <int NORB, typename WT>
__global__ __launch_bounds__(NTMAX, kWaves) void nos_kernel(FwdArgs a) {
  __shared__ SplineShared<NORB> sh;
  const int b = blockIdx.x;
  const int unit = (b % NXCD) * a.per_xcd + b / NXCD;  // XCD-aware: contiguous tiles per XCD
  if (unit >= a.nunits) return;
  spline_unit<NORB, WT, 3>(a, unit, sh);
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
