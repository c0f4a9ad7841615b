// What the spline kernels share (gfx950): the tile of a work unit and its layout in LDS, the steps of a grid
// point's sums (tetra_spline.h), the running sums. Internal header.
#pragma once

#include "tetra_device.h"
#include "tetra_forward_args.h"
#include "tetra_spline.h"
#include "tetra_wave.h"

namespace tetra {

constexpr int kSide = 8;                  // largest tile side, in cubes
constexpr int NTMAX = kSide * kSide * kSide;  // lanes of the largest workgroup: one per cube
constexpr int NWMAX = NTMAX / 64;
constexpr int PZ = kSide + 1, PY = PZ * PZ;   // strides of the tile's grid points along axes 2 and 1
constexpr int NP = PZ * PZ * PZ;
// Two workgroups of eight waves per CU: four waves per SIMD, 80 KB of LDS each.
constexpr int kWaves = 4;
constexpr int kLdsBytes = 81920;
constexpr int NXCD = 8;

constexpr int kQueue = 512;     // tetrahedra of a unit that are queued for the sum energy by energy
constexpr int kLongRows = 256;  // energies from which on two lanes share a tetrahedron

constexpr int SZ = PZ + 1, SY = PZ * SZ + SZ;     // strides of the knots, a far one at the end of every line and plane
constexpr int kKnotMargin = SY + SZ + 1;        // the furthest neighbour offset
constexpr int kKnotPad = PZ * SY + 2 * kKnotMargin;
constexpr int kWeightPad = PY + PZ + 1;         // words before and after the weights that neighbour offsets reach

// Global float add without a compare-and-swap loop (device memory from hipMalloc).
__device__ __forceinline__ void atomic_add_global(float* p, float v) { unsafeAtomicAdd(p, v); }

__device__ __forceinline__ int wrap(int v, int n) {
  if (v >= n) v -= n;
  if (v >= n) v %= n;
  return v;
}

// Tile of a work unit: first cube and number of cubes along each axis (the grid's sides are dealt to the
// tiles as evenly as they go).
struct Tile {
  int x0, y0, z0, cx, cy, cz;
};
__device__ __forceinline__ int divide(uint32_t n, FastDiv d) { return (int)(((uint64_t)n * d.m) >> d.s); }
__device__ __forceinline__ Tile unit_tile(const FwdArgs& a, int unit, int& band) {
  band = divide(unit, a.by_ntiles);
  const int tile = unit - band * a.ntiles;
  const int r = divide(tile, a.by_t3), tz = tile - r * a.t3;
  const int tx = divide(r, a.by_t2), ty = r - tx * a.t2;
  Tile t;
  t.x0 = tx * a.s1 + min(tx, a.r1);
  t.cx = a.s1 + (tx < a.r1);
  t.y0 = ty * a.s2 + min(ty, a.r2);
  t.cy = a.s2 + (ty < a.r2);
  t.z0 = tz * a.s3 + min(tz, a.r3);
  t.cz = a.s3 + (tz < a.r3);
  return t;
}

// q / d for q < 1024 and uniform d <= 9 by a multiplication (inv = small_inverse(d), 65536 / d + 1 without the vector
// division that stands at the start of a unit otherwise).
__device__ __forceinline__ int small_inverse(int d) {
  int inv = 65537;
#pragma unroll
  for (int i = 2; i <= kSide + 1; ++i) inv = d == i ? 65536 / i + 1 : inv;
  return inv;
}
__device__ __forceinline__ int small_div(int q, int inv) { return (q * inv) >> 16; }

// 1 / (u_q - u0) of a knot's neighbours in the layout of the knots.
__device__ __forceinline__ void knot_reciprocals(const double* up, double u0, double M[kNeighbours]) {
#pragma unroll
  for (int u = 0; u < kNeighbours; ++u) {
    int dx, dy, dz;
    neighbour_offset(u, dx, dy, dz);
    M[u] = up[dx * SY + dy * SZ + dz] - u0;
  }
#pragma unroll
  for (int u = 0; u < kNeighbours; ++u) {
    M[u] = rcp64(M[u]);
    if (u % 7 == 6) schedule_fence();  // a few at a time: fewer registers
  }
}

// sum_u M_u (b_u - b_p) from the point's place in an orbital's weights and Ms = sum_u M_u.
__device__ __forceinline__ double knot_contract(const double M[kNeighbours], double Ms, const float* w) {
  double Q = -Ms * (double)w[0], Q1 = 0.0;
#pragma unroll
  for (int u = 0; u < kNeighbours; ++u) {
    int dx, dy, dz;
    neighbour_offset(u, dx, dy, dz);
    double& q = (u & 1) ? Q1 : Q;
    q = __builtin_fma(M[u], (double)w[dx * PY + dy * PZ + dz], q);
  }
  return Q + Q1;
}

// Copies of a histogram plane, a power of two up to 32, as the LDS left over allows: with few rows the lanes of a wave
// share bins. 64^3 x 8 x 8 x 50, 100, 200, 1000: 0.226, 0.214, 0.189, 0.167 ms with up to four copies of an even
// stride, 0.159, 0.165, 0.171, 0.167 ms with these; 48 x 32 x 30 x 16 x 16 x 51: 0.227 -> 0.114 ms.
__device__ __forceinline__ int histogram_copies(int plane, int words) {
  int copies = 1;
  while (copies < 32 && 2 * copies * plane <= words) copies *= 2;
  return copies;
}

// Four running sums down each of the gm columns (RS words) of a histogram of `copies` planes, 128 rows at a
// time; the result is in the first plane, the others are cleared on demand. A row more than there are is read and written at most.
template <typename Acc>
__device__ __forceinline__ void running_sums(Acc* hist, int gm, int RS, int plane, int copies, int rows,
                                             bool clear = false) {
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));  // nothing formed from it is kept live from one group of orbitals to the next
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int NW = blockDim.x >> 6;
  for (int m = wave; m < gm; m += NW) {
    Acc c[4] = {Acc(0), Acc(0), Acc(0), Acc(0)};
    for (int r0 = 0; r0 < rows; r0 += 128) {
      const int r = r0 + 2 * lane;
      Acc* hm = hist + m * RS + r;
      Acc v0 = Acc(0), v1 = Acc(0);
      if (r < rows)
        for (int k = 0; k < copies; ++k) {
          v0 += hm[k * plane];
          v1 += hm[k * plane + 1];
          if (clear) hm[k * plane] = hm[k * plane + 1] = Acc(0);
        }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        v1 += v0;
        const Acc t = wave_scan(v1) + c[k];
        c[k] = last_lane(t);
        v0 += t - v1;
        v1 = t;
      }
      if (r < rows) {
        hm[0] = v0;
        hm[1] = v1;
      }
    }
  }
}

// put(j, g) with the corner weights dw/dE of a tetrahedron (sorted corner energies e) at every step-th
// energy of its window in [lo, hi], from the first-th on.
template <typename F>
__device__ __forceinline__ void tet_energies(const float e[4], const FwdArgs& a, int lo, int hi, int first, int step,
                                             F&& put) {
  int jlo, jhi;
  energy_window(e[0], e[3], a.e0, a.inv_de, lo, hi, jlo, jhi);
  const TetSetup cs = tet_setup(e, a.e0, a.V);
  tet_window(cs, a.de, lo, hi, jlo, jhi);
  int jA, jB;
  case_split(cs, a.de, a.inv_de, jlo, jhi, jA, jB);
  float coef[4][4];
  if (jB > jA) corner_dos_B_coeffs(cs, a.V, coef);
  for (int j = jlo + first; j <= jhi; j += step) {
    float g[4];
    if (j <= jA) corner_dos_A(cs, local_x(cs, j, a.de), g);
    else if (j <= jB) corner_dos_B_poly(coef, local_z(cs, j, a.de), g);
    else corner_dos_C(cs, local_y(cs, j, a.de), g);
    put(j, g);
  }
}

}  // namespace tetra
