// Susceptibility kernel: orbital-resolved imaginary part of the bare (Lindhard) susceptibility at zero
// temperature for a transfer q on the k-grid, as the spectral weight S_m(q, w) of tetra_chi_device.h
// (Im chi_0 = -pi S), by the linear tetrahedron method of Guterding & Jeschke (arXiv:1710.10789,
// Sec. II) with the difference energy eps_n'(k + q) - eps_n(k) in the role of the band energy.
//
// Two passes over the band pairs (n, n'), which add into the same output:
//  * chi_spline_kernel (tetra_chi_spline_kernels.h): the tetrahedra that are occupied in one band and empty in the
//    other at every corner, most of them, in the spline form of the DOS;
//  * chi_kernel, here: the tetrahedra that E_F cuts in one of the bands.
// One workgroup per (tile of TX x TY x TZ cubes, band n), or several, each with a share of the bands n', tile-major,
// and each XCD takes a contiguous range of them. For a pair the tile's grid points are staged in LDS with eps_n at
// the point and eps_n' at the point shifted by q (periodic); every lane goes over the six tetrahedra of Table I of
// its cube and queues the occupation regions that have to be clipped; only then the product weights
// W_m = b_mn(k) b_mn'(k + q) are staged. Each energy pass lists the regions' pieces (a region is clipped at eps = E_F
// and eps' = E_F into at most nine sub-tetrahedra, held as barycentric rows in the parent), then every lane takes
// pieces: the DOS of eps' - eps on each with W formed at its vertices and its share of the volume (sort, exact window,
// case split, corner weights of Sec. II.C).
// The LDS histograms hold fixed point with a power-of-two scale from a bound: the part of a
// tetrahedron on either side of an occupation boundary has a section no larger than the whole
// tetrahedron's, so a tetrahedron adds at most 12 V max|W| / (max - min of eps' - eps) to any bin
// (V = V_T/(4 V_G)). With non-negative weights each region's terms are non-negative: one histogram per
// region, two orbitals per 64-bit word; otherwise one signed 64-bit histogram. The sums are exact
// integers, so the order in which the queue is filled and worked off does not change them. One global
// float atomic per touched (energy, orbital) bin at the end.
//
// 64^3 x 8 x 8 x 500: 1.72 ms when one kernel took both kinds of region (every tetrahedron's window energy by
// energy), 1.40 ms now, 0.73 ms of it the spline pass and 0.65 ms this kernel's, bound by instruction issue: of that
// about 0.13 ms staging and the search for regions, 0.06 ms weights, 0.17 ms listing the pieces and clearing and
// flushing the histogram, 0.3 ms clipping and summing the pieces. Leaving the pieces in nine slots per region, two
// or three of them filled, took 0.1 ms more, and workgroups for pairs that E_F cuts in neither band 0.15 ms.

#include <algorithm>
#include <type_traits>

#include "tetra_chi_args.h"
#include "tetra_chi_device.h"
#include "tetra_device.h"
#include "tetra_internal.h"
#include "tetra_wave.h"
#include "tetra_weights.h"

namespace tetra {

namespace {

constexpr int NT = kTileCubes;
constexpr int NPMAX = kTilePointsMax;
constexpr int QCAP = NT * 12 + 576;  // queue: the most regions a tile has, and the pieces of 64 of them
constexpr int HCAP = 2048;  // LDS histogram capacity in 64-bit words
constexpr int NXCD = 8;

struct ChiArgs {
  const float* eps;
  const void* w;
  const float* w_scale;
  float* out;
  int n1, n2, n3, nb, ne;
  int q1, q2, q3;  // transfer in grid steps, reduced to [0, n)
  float ef, e0, de, inv_de, V;
  int TX, TY, TZ;
  int t1, t2, t3, ntiles;
  int parts, nunits, per_xcd;  // workgroups per (tile, band n), in all, per XCD
  // Energy range (smallest, largest finite value) of every (tile, band): rows [0, nb) at the tile's
  // points, rows [nb, 2 nb) at the points shifted by q; NULL where not computed.
  const float2* ranges;
};

__device__ __forceinline__ int wrap_index(int v, int n) {
  if (v >= n) v -= n;
  if (v >= n) v %= n;
  return v;
}

// First pass of the workspace variant: one workgroup per (tile, band) writes the band's energy range
// over the tile's grid points (the points a unit stages) and over the same points shifted by q.
__global__ __launch_bounds__(NT) void chi_ranges_kernel(ChiArgs a) {
  __shared__ float s_r[4 * (NT / 64)];
  const int tile = blockIdx.x % a.ntiles, band = blockIdx.x / a.ntiles;
  const int PY = a.TY + 1, PZ = a.TZ + 1, NP = (a.TX + 1) * PY * PZ;
  const int tz = tile % a.t3, ty = (tile / a.t3) % a.t2, tx = tile / (a.t3 * a.t2);
  const int x0 = tx * a.TX, y0 = ty * a.TY, z0 = tz * a.TZ;
  const int64_t nk = (int64_t)a.n1 * a.n2 * a.n3;
  const float* e_b = a.eps + (int64_t)band * nk;
  float kmin = __builtin_huge_valf(), kmax = -__builtin_huge_valf(), qmin = kmin, qmax = kmax;
  for (int p = threadIdx.x; p < NP; p += NT) {
    const int pz = p % PZ, py = (p / PZ) % PY, px = p / (PZ * PY);
    const int i1 = wrap_index(x0 + px, a.n1), i2 = wrap_index(y0 + py, a.n2), i3 = wrap_index(z0 + pz, a.n3);
    const float e = e_b[((int64_t)i1 * a.n2 + i2) * a.n3 + i3];
    const float eq = e_b[((int64_t)wrap_index(i1 + a.q1, a.n1) * a.n2 + wrap_index(i2 + a.q2, a.n2)) * a.n3 +
                         wrap_index(i3 + a.q3, a.n3)];
    if (__builtin_isfinite(e)) {
      kmin = fminf(kmin, e);
      kmax = fmaxf(kmax, e);
    }
    if (__builtin_isfinite(eq)) {
      qmin = fminf(qmin, eq);
      qmax = fmaxf(qmax, eq);
    }
  }
  kmin = wave_min(kmin);
  kmax = wave_max(kmax);
  qmin = wave_min(qmin);
  qmax = wave_max(qmax);
  if ((threadIdx.x & 63) == 0) {
    const int wv = threadIdx.x >> 6;
    s_r[wv] = kmin;
    s_r[(NT / 64) + wv] = kmax;
    s_r[2 * (NT / 64) + wv] = qmin;
    s_r[3 * (NT / 64) + wv] = qmax;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int wv = 1; wv < NT / 64; ++wv) {
      kmin = fminf(kmin, s_r[wv]);
      kmax = fmaxf(kmax, s_r[(NT / 64) + wv]);
      qmin = fminf(qmin, s_r[2 * (NT / 64) + wv]);
      qmax = fmaxf(qmax, s_r[3 * (NT / 64) + wv]);
    }
    float2* r = const_cast<float2*>(a.ranges);
    r[(int64_t)band * a.ntiles + tile] = make_float2(kmin, kmax);
    r[(int64_t)(a.nb + band) * a.ntiles + tile] = make_float2(qmin, qmax);
  }
}

// Waves per SIMD the kernel is held to: 88-128 VGPRs up to 8 orbitals, 133-168 up to 14, 183-189 above (at 3 waves 20 to
// 44 bytes of scratch; 40^3 x 16 x 16 x 300, both passes, 1.67 and 1.64 ms at 3 and 2). No vector registers spilled.
constexpr int chi_waves(int norb) { return norb <= 8 ? 4 : norb <= 14 ? 3 : 2; }

// Whether E_F cuts one of the two bands: without, every region is a whole tetrahedron or empty.
__device__ __forceinline__ bool crosses(float emin, float emax, float pmin, float pmax, float ef) {
  return (emin < ef && emax > ef) || (pmin < ef && pmax > ef);
}

template <int NORB>
struct ChiShared {
  float e[NPMAX];
  float ep[NPMAX];
  float W[NPMAX * NORB];
  unsigned long long hist[HCAP];
  float red[8 * (NT / 64)];
  // regions to clip: lane of the cube << 4 | tetrahedron << 1 | region (at most 6 x 2 per cube); after them the
  // pieces of some: place of the region << 4 | first piece << 2 | second piece
  unsigned short q[QCAP];
  int qn, pn;
};

// The pair of bands (n, np) over a tile; every lane of the workgroup calls it.
template <int NORB, typename WT>
__device__ __forceinline__ void chi_unit(const ChiArgs& a, int tile, int n, int np, ChiShared<NORB>& sh) {
  constexpr int RS = (HCAP / NORB - 1) | 1;  // histogram row stride (one row per orbital), odd
  float *const s_e = sh.e, *const s_ep = sh.ep, *const s_W = sh.W, *const s_red = sh.red;
  unsigned long long* const s_hist = sh.hist;
  unsigned short* const s_q = sh.q;
  int &s_qn = sh.qn, &s_pn = sh.pn;
  const int TX = a.TX, TY = a.TY, TZ = a.TZ;
  const int PY = TY + 1, PZ = TZ + 1;
  const int NP = (TX + 1) * PY * PZ;
  const int tz = tile % a.t3;
  const int ty = (tile / a.t3) % a.t2;
  const int tx = tile / (a.t3 * a.t2);
  const int x0 = tx * TX, y0 = ty * TY, z0 = tz * TZ;
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));  // nothing formed from it is kept live from one pair to the next
  const int64_t nk = (int64_t)a.n1 * a.n2 * a.n3;
  const float* eps_n = a.eps + (int64_t)n * nk;
  const float* eps_p = a.eps + (int64_t)np * nk;
  const WT* w_n = static_cast<const WT*>(a.w) + (int64_t)n * NORB * nk;
  const WT* w_p = static_cast<const WT*>(a.w) + (int64_t)np * NORB * nk;
  const float sc_n = a.w_scale ? a.w_scale[n] : 1.0f, sc_p = a.w_scale ? a.w_scale[np] : 1.0f;

  // Stage the tile's energies: eps_n at the point, eps_n' at the point + q; reduce the ranges of eps,
  // eps' and eps' - eps. Most (tile, band pair) units end here: no region can be occupied on one side
  // and empty on the other, or eps' - eps stays outside the energy grid; their weights are never read.
  auto point_k = [&](int p, int64_t& k, int64_t& kq) {
    const int pz = p % PZ, py = (p / PZ) % PY, px = p / (PZ * PY);
    const int i1 = wrap_index(x0 + px, a.n1), i2 = wrap_index(y0 + py, a.n2), i3 = wrap_index(z0 + pz, a.n3);
    k = ((int64_t)i1 * a.n2 + i2) * a.n3 + i3;
    kq = ((int64_t)wrap_index(i1 + a.q1, a.n1) * a.n2 + wrap_index(i2 + a.q2, a.n2)) * a.n3 +
         wrap_index(i3 + a.q3, a.n3);
  };
  if (tid == 0) s_qn = 0;
  float r_emin = __builtin_huge_valf(), r_emax = -__builtin_huge_valf();
  float r_pmin = __builtin_huge_valf(), r_pmax = -__builtin_huge_valf();
  float r_dmin = __builtin_huge_valf(), r_dmax = -__builtin_huge_valf();
  for (int p = tid; p < NP; p += NT) {
    int64_t k, kq;
    point_k(p, k, kq);
    const float e = eps_n[k], ep = eps_p[kq];
    s_e[p] = e;
    s_ep[p] = ep;
    if (__builtin_isfinite(e) && __builtin_isfinite(ep)) {
      r_emin = fminf(r_emin, e);
      r_emax = fmaxf(r_emax, e);
      r_pmin = fminf(r_pmin, ep);
      r_pmax = fmaxf(r_pmax, ep);
      r_dmin = fminf(r_dmin, ep - e);
      r_dmax = fmaxf(r_dmax, ep - e);
    }
  }
  float red[8] = {wave_min(r_emin), wave_max(r_emax), wave_min(r_pmin), wave_max(r_pmax),
                  wave_min(r_dmin), wave_max(r_dmax), 0.0f, 0.0f};
  if ((tid & 63) == 0)
#pragma unroll
    for (int i = 0; i < 6; ++i) s_red[i * (NT / 64) + (tid >> 6)] = red[i];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    float v = s_red[i * (NT / 64)];
#pragma unroll
    for (int wv = 1; wv < NT / 64; ++wv) {
      const float x = s_red[i * (NT / 64) + wv];
      v = (i == 0 || i == 2 || i == 4) ? fminf(v, x) : fmaxf(v, x);
    }
    red[i] = v;
  }
  const float ef = a.ef;
  if (!(red[4] <= red[5])) return;  // no finite pair in this tile (uniform across the block)
  if (!region_possible(0, red[0], red[1], red[2], red[3], ef) && !region_possible(1, red[0], red[1], red[2], red[3], ef))
    return;
  int J0, J1;
  range_window(red[4], red[5], a.e0, a.inv_de, a.ne, J0, J1);
  if (J0 > J1) return;
  if (!crosses(red[0], red[1], red[2], red[3], ef)) return;

  // First point of lane i's cube; false where the grid ends before it.
  auto lane_cube = [&](int i, int& pbase) {
    const int cz = i % TZ, cy = (i / TZ) % TY, cx = i / (TZ * TY);
    pbase = (cx * PY + cy) * PZ + cz;
    return cx < TX && (x0 + cx < a.n1) && (y0 + cy < a.n2) && (z0 + cz < a.n3);
  };
  auto point_offset = [PY, PZ](int s) { return (s & 1) * (PY * PZ) + ((s >> 1) & 1) * PZ + (s >> 2); };

  // The regions of tetrahedron t of this lane's cube that are to be clipped, and the range of eps' - eps over it;
  // false when there is none that can contribute to [lo, hi]. A region that is the whole tetrahedron (n occupied
  // and n' empty at every corner for region 0, the reverse for region 1) is the spline pass's.
  auto regions = [&](int pbase, int t, int lo, int hi, bool reg[2], float& dmin, float& dmax) {
    const uint32_t slots = tet_slots(t);
    float emin = __builtin_huge_valf(), emax = -emin, pmin = emin, pmax = -emin;
    dmin = emin;
    dmax = -emin;
    bool fin = true;
#pragma unroll
    for (int l = 0; l < 4; ++l) {
      const int p = pbase + point_offset((slots >> (4 * l)) & 7);
      const float e = s_e[p], ep = s_ep[p];
      fin = fin && __builtin_isfinite(e) && __builtin_isfinite(ep);
      emin = fminf(emin, e);
      emax = fmaxf(emax, e);
      pmin = fminf(pmin, ep);
      pmax = fmaxf(pmax, ep);
      dmin = fminf(dmin, ep - e);
      dmax = fmaxf(dmax, ep - e);
    }
    if (!fin || !(dmax > dmin)) return false;
    const int whole = (emax <= ef && pmin >= ef) ? 0 : (emin >= ef && pmax <= ef) ? 1 : -1;
    reg[0] = whole != 0 && region_possible(0, emin, emax, pmin, pmax, ef);
    reg[1] = whole != 1 && region_possible(1, emin, emax, pmin, pmax, ef);
    if (!reg[0] && !reg[1]) return false;
    int jlo, jhi;
    energy_window(dmin, dmax, a.e0, a.inv_de, lo, hi, jlo, jhi);
    return jlo <= jhi + 2;
  };

  // The regions to clip into the queue, every lane on its own cube. They lie where a band crosses E_F, in a few
  // cubes of the tile; shared out over all lanes they do not hold one wavefront, and the workgroup behind its
  // barrier, for the whole pass. With them a bound on any bin's |sum|: sum over their tetrahedra of 12 V max|W| /
  // (dmax - dmin), 12 V max|W| below, and the range of eps' - eps. Narrow tetrahedra (a range below 2 de) give
  // spikes that make B loose.
  float bound = 0.0f, narrow = 0.0f, lo = __builtin_huge_valf(), hi = -__builtin_huge_valf();
  if (int pbase; lane_cube(tid, pbase)) {
#pragma unroll 1
    for (int t = 0; t < 6; ++t) {
      bool reg[2];
      float dmin, dmax;
      if (!regions(pbase, t, J0, J1, reg, dmin, dmax)) continue;
#pragma unroll
      for (int r = 0; r < 2; ++r)
        if (reg[r]) s_q[atomicAdd(&s_qn, 1)] = (unsigned short)((tid << 4) | (t << 1) | r);
      const float term = rcp(dmax - dmin);
      bound += term;
      if (dmax - dmin < 2.0f * a.de) narrow += term;
      lo = fminf(lo, dmin);
      hi = fmaxf(hi, dmax);
    }
  }
  bound = wave_sum(bound);
  narrow = wave_sum(narrow);
  lo = wave_min(lo);
  hi = wave_max(hi);
  __syncthreads();  // every lane has read s_red
  if ((tid & 63) == 0) {
    s_red[tid >> 6] = bound;
    s_red[(NT / 64) + (tid >> 6)] = narrow;
    s_red[2 * (NT / 64) + (tid >> 6)] = lo;
    s_red[3 * (NT / 64) + (tid >> 6)] = hi;
  }
  __syncthreads();
  float B = 0.0f, Bn = 0.0f;
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) {
    B += s_red[i];
    Bn += s_red[NT / 64 + i];
    lo = fminf(lo, s_red[2 * (NT / 64) + i]);
    hi = fmaxf(hi, s_red[3 * (NT / 64) + i]);
  }
  if (!(B > 0.0f)) return;  // nothing to clip (uniform across the block)
  range_window(lo, hi, a.e0, a.inv_de, a.ne, J0, J1);
  J0 = uniform(J0);
  J1 = uniform(J1);

  // The weights W = b_n(k) b_n'(k + q), with the largest |W| and the smallest W.
  float r_wmax = 0.0f, r_wmin = 0.0f;
  for (int p = tid; p < NP; p += NT) {
    int64_t k, kq;
    point_k(p, k, kq);
#pragma unroll
    for (int m = 0; m < NORB; ++m) {
      const float W = weight_value(w_n[(int64_t)m * nk + k], sc_n) * weight_value(w_p[(int64_t)m * nk + kq], sc_p);
      s_W[p * NORB + m] = W;
      r_wmax = fmaxf(r_wmax, fabsf(W));
      r_wmin = fminf(r_wmin, W);
    }
  }
  r_wmax = wave_max(r_wmax);
  r_wmin = wave_min(r_wmin);
  if ((tid & 63) == 0) {
    s_red[6 * (NT / 64) + (tid >> 6)] = r_wmax;
    s_red[7 * (NT / 64) + (tid >> 6)] = r_wmin;
  }
  __syncthreads();
  red[6] = s_red[6 * (NT / 64)];
  red[7] = s_red[7 * (NT / 64)];
#pragma unroll
  for (int wv = 1; wv < NT / 64; ++wv) {
    red[6] = fmaxf(red[6], s_red[6 * (NT / 64) + wv]);
    red[7] = fminf(red[7], s_red[7 * (NT / 64) + wv]);
  }
  const float wmax = red[6], wmin = red[7];

  const float c12 = 12.0f * a.V * wmax;
  B = fminf(B * c12, 3.0e38f);
  Bn = fminf(Bn * c12, 3.0e38f);
  if (!(B > 0.0f)) return;
  // Packed: within one region every contribution is non-negative when the weights are (corner weights
  // and barycentric coordinates are), so each region gets a histogram of its own with two orbitals per
  // 64-bit word as 32-bit fields (B S <= 2^30, no carry between fields) and the result is their
  // difference. Otherwise one signed 64-bit histogram (B S <= 2^62).
  const bool packed = wmin >= 0.0f && Bn <= 0.5f * B;  // uniform across the block
  int bexp;
  frexpf(fminf(B, 3.0e38f), &bexp);  // B <= 2^bexp
  const int sexp = uniform(min((packed ? 30 : 62) - bexp, 126));
  const float VS = uniform(a.V * ldexpf(1.0f, sexp));  // V_T/(4 V_G) in units of the fixed point

  auto passes = [&](auto packed_tag) {
    constexpr bool PACKED = decltype(packed_tag)::value;
    constexpr int NPAIR = (NORB + 1) / 2;
    // rows: packed, one per orbital pair in each region's half of the histogram; wide, one per orbital
    constexpr int RSP = (HCAP / 2 / NPAIR - 1) | 1;
    constexpr int RSX = PACKED ? RSP : RS;
    unsigned long long* hist_m = s_hist + (PACKED ? HCAP / 2 : 0);  // region -1 (packed only)
    // Corner weights dw/dE of a (sub-)tetrahedron's sorted vertices at grid energy j.
    auto corner_g = [&](const TetSetup& cs, const float (&coef)[4][4], int j, int jA, int jB, float g[4]) {
      if (j <= jA) {
        corner_dos_A(cs, local_x(cs, j, a.de), g);
        g[0] = fmaxf(g[0], 0.0f);
      } else if (j <= jB) {
        corner_dos_B_poly(coef, local_z(cs, j, a.de), g);
#pragma unroll
        for (int l = 0; l < 4; ++l) g[l] = fmaxf(g[l], 0.0f);
      } else {
        corner_dos_C(cs, local_y(cs, j, a.de), g);
        g[3] = fmaxf(g[3], 0.0f);
      }
    };
    // One energy's terms sum_l G_l Wr[l][m] into the region's histogram row h.
    auto deposit = [&](unsigned long long* h, float G[4], const float (&Wr)[4][NORB], float sign) {
      if (PACKED) {
        // non-negative terms: the truncating conversion of 1/2 + v rounds (halves up)
#pragma unroll
        for (int pr = 0; pr < NPAIR; ++pr) {
          const int m0 = 2 * pr, m1 = 2 * pr + 1;
          const float v0 = __builtin_fmaf(G[0], Wr[0][m0], __builtin_fmaf(G[1], Wr[1][m0],
                           __builtin_fmaf(G[2], Wr[2][m0], __builtin_fmaf(G[3], Wr[3][m0], 0.5f))));
          unsigned long long word = (unsigned long long)(unsigned)v0;
          if (m1 < NORB) {
            const float v1 = __builtin_fmaf(G[0], Wr[0][m1], __builtin_fmaf(G[1], Wr[1][m1],
                             __builtin_fmaf(G[2], Wr[2][m1], __builtin_fmaf(G[3], Wr[3][m1], 0.5f))));
            word |= (unsigned long long)(unsigned)v1 << 32;
          }
          atomicAdd(&h[pr * RSX], word);
        }
      } else {
#pragma unroll
        for (int l = 0; l < 4; ++l) G[l] *= sign;
#pragma unroll
        for (int m = 0; m < NORB; ++m) {
          const float v = __builtin_fmaf(G[0], Wr[0][m], __builtin_fmaf(G[1], Wr[1][m],
                                         __builtin_fmaf(G[2], Wr[2][m], G[3] * Wr[3][m])));
          atomicAdd(&h[m * RSX], (unsigned long long)__float2ll_rn(v));
        }
      }
    };
    for (int c0 = J0; c0 <= J1; c0 += RSX) {
      const int c1 = min(c0 + RSX - 1, J1);
      const int L = c1 - c0 + 1;
      int tid = threadIdx.x;  // opaque again: the addresses formed from it are formed in each pass
      asm volatile("" : "+v"(tid));
      const int rows = PACKED ? NPAIR : NORB;
      for (int q = tid; q < rows * L; q += NT) {
        const int m = q / L;
        s_hist[m * RSX + (q - m * L)] = 0ull;
        if (PACKED) hist_m[m * RSX + (q - m * L)] = 0ull;
      }
      __syncthreads();
      // The queued regions, clipped at the two occupation boundaries into at most 3 x 3 sub-tetrahedra, as many
      // regions at a time as the rest of the queue holds pieces for. First the pieces are listed, a lane per
      // (first piece, region), so that every lane then has a piece: of nine slots per region two or three hold
      // one, spread over all of a wavefront's slots. Each piece redoes its region's planes and first
      // clipping from LDS (nothing of the clipping stays live over a piece's energy loop).
      const int nq = s_qn, most = (QCAP - nq) / 9;
      constexpr float I[4][4] = {{1.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 1.0f, 0.0f, 0.0f},
                                 {0.0f, 0.0f, 1.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 1.0f}};
      // A region's corners: their difference energies dd, points q and occupation planes (f1, f2c <= 0 inside).
      auto region = [&](int item, float dd[4], int q[4], float f1[4], float f2c[4]) {
        const int it = item >> 4, t = (item >> 1) & 7, r = item & 1;
        const int qz = it % TZ, qy = (it / TZ) % TY, qx = it / (TZ * TY);
        const int qbase = (qx * PY + qy) * PZ + qz;
        const uint32_t slots = tet_slots(t);
        float er[4], epr[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          q[c] = qbase + point_offset((slots >> (4 * c)) & 7);
          er[c] = s_e[q[c]];
          epr[c] = s_ep[q[c]];
        }
        region_planes(r, er, epr, ef, f1, f2c);
#pragma unroll
        for (int c = 0; c < 4; ++c) dd[c] = epr[c] - er[c];
        return (f1[0] <= 0.0f) + (f1[1] <= 0.0f) + (f1[2] <= 0.0f) + (f1[3] <= 0.0f);
      };
      // Vertices A of its piece ia and the second plane f2 at them. The corners are reordered so that those inside
      // the first plane come first: the clipping then starts from the identity, whose unit rows fold into constants.
      auto first_piece = [&](int ni1, int ia, float dd[4], int q[4], float f1[4], float f2c[4], float A[4][4],
                             float f2[4]) {
        if (ni1 > 0 && ni1 < 4) inside_first_corners(f1, f2c, dd, q);
        clip_piece(I, f1, ni1, ia, A);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          f2[i] = __builtin_fmaf(A[i][0], f2c[0], __builtin_fmaf(A[i][1], f2c[1],
                                 __builtin_fmaf(A[i][2], f2c[2], A[i][3] * f2c[3])));
        return (f2[0] <= 0.0f) + (f2[1] <= 0.0f) + (f2[2] <= 0.0f) + (f2[3] <= 0.0f);
      };
#pragma unroll 1
      for (int i0 = 0; i0 < nq; i0 += most) {
      const int nr = min(most, nq - i0);
      if (tid == 0) s_pn = 0;
      __syncthreads();
#pragma unroll 1
      for (int ip = tid; ip < 3 * nr; ip += NT) {
        const int ia = (ip >= nr) + (ip >= 2 * nr), iq = i0 + ip - ia * nr;
        float dd[4], A[4][4], f1[4], f2[4], f2c[4];
        int q[4];
        const int ni1 = region(s_q[iq], dd, q, f1, f2c);
        if (ia >= clip_pieces(ni1)) continue;
        const int count = clip_pieces(first_piece(ni1, ia, dd, q, f1, f2c, A, f2));
        unsigned short* to = &s_q[nq + atomicAdd(&s_pn, count)];
        for (int ib = 0; ib < count; ++ib) to[ib] = (unsigned short)(iq << 4 | ia << 2 | ib);
      }
      __syncthreads();
      const int pieces = s_pn;
#pragma unroll 1
      for (int ip = tid; ip < pieces; ip += NT) {
        const int entry = s_q[nq + ip], ia = (entry >> 2) & 3, ib = entry & 3, item = s_q[entry >> 4], r = item & 1;
        float dd[4], A[4][4], f1[4], f2[4], f2c[4];
        int q[4];
        const int ni1 = region(item, dd, q, f1, f2c);
        if (ia >= clip_pieces(ni1)) continue;
        const int ni2 = first_piece(ni1, ia, dd, q, f1, f2c, A, f2);
        if (ib >= clip_pieces(ni2)) continue;
        if (ni2 > 0 && ni2 < 4) inside_first(A, f2);
        float S[4][4];
        clip_piece(A, f2, ni2, ib, S);
        const float frac = sub_volume(S);
        if (!(frac > 0.0f)) continue;
        float d[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
          d[i] = __builtin_fmaf(S[i][0], dd[0], __builtin_fmaf(S[i][1], dd[1],
                                __builtin_fmaf(S[i][2], dd[2], S[i][3] * dd[3])));
        sort4_rows(d, S);
        int jlo, jhi;
        energy_window(d[0], d[3], a.e0, a.inv_de, c0, c1, jlo, jhi);
        if (jlo > jhi + 2) continue;
        const float Vs = VS * frac;
        const TetSetup cs = tet_setup(d, a.e0, Vs);
        tet_window(cs, a.de, c0, c1, jlo, jhi);
        if (jlo > jhi) continue;
        // W at the sorted vertices (linear on the parent): Wv[l] = sum_c S[l][c] W_c
        float wv[4][NORB];
#pragma unroll
        for (int l = 0; l < 4; ++l)
#pragma unroll
          for (int m = 0; m < NORB; ++m) wv[l][m] = 0.0f;
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
          for (int m = 0; m < NORB; ++m) {
            const float wc = s_W[q[c] * NORB + m];
#pragma unroll
            for (int l = 0; l < 4; ++l) wv[l][m] = __builtin_fmaf(S[l][c], wc, wv[l][m]);
          }
        int jA, jB;
        case_split(cs, a.de, a.inv_de, jlo, jhi, jA, jB);
        float coef[4][4];
        if (jB > jA) corner_dos_B_coeffs(cs, Vs, coef);
        const float sign = r == 0 ? 1.0f : -1.0f;
        unsigned long long* hreg = (PACKED && r == 1) ? hist_m : s_hist;
        for (int j = jlo; j <= jhi; ++j) {
          float g[4];
          corner_g(cs, coef, j, jA, jB, g);
          deposit(&hreg[j - c0], g, wv, sign);
        }
      }
      __syncthreads();
      }
      for (int q = tid; q < L * NORB; q += NT) {
        const int rr = q / NORB, m = q - rr * NORB;
        double v;
        if (PACKED) {
          const unsigned long long wp = s_hist[(m >> 1) * RSX + rr], wm = hist_m[(m >> 1) * RSX + rr];
          const unsigned fp = (m & 1) ? (unsigned)(wp >> 32) : (unsigned)(wp & 0xffffffffull);
          const unsigned fm = (m & 1) ? (unsigned)(wm >> 32) : (unsigned)(wm & 0xffffffffull);
          v = (double)fp - (double)fm;
        } else {
          v = (double)(long long)s_hist[m * RSX + rr];
        }
        if (v != 0.0) unsafeAtomicAdd(&a.out[(int64_t)(c0 + rr) * NORB + m], (float)ldexp(v, -sexp));
      }
      __syncthreads();
    }
  };
  if (packed)
    passes(std::true_type{});
  else
    passes(std::false_type{});
}

// A workgroup takes every parts-th of the bands n' that can contribute with its band n over its tile. With the
// first pass's ranges the others cost nothing: the table's ranges bound the staged values (they include points
// where only one band is finite), so its tests only ever let through pairs that the unit's own then drop.
template <int NORB, typename WT>
__global__ __launch_bounds__(NT, chi_waves(NORB)) void chi_kernel(ChiArgs a) {
  __shared__ ChiShared<NORB> sh;
  const int b = blockIdx.x;
  const int unit = (b % NXCD) * a.per_xcd + b / NXCD;  // tile-major: the tile's points stay in the XCD's L2
  if (unit >= a.nunits) return;
  const int per_tile = a.nb * a.parts, tile = unit / per_tile, r = unit - tile * per_tile;
  const int n = r / a.parts, part = r - n * a.parts;
  int k = 0;
  for (int n0 = 0; n0 < a.nb; n0 += 64) {
    int lane = threadIdx.x;
    asm volatile("" : "+v"(lane));
    const int np = n0 + (lane & 63);
    bool can = np < a.nb;
    if (can && a.ranges) {
      const float2 rk = a.ranges[(int64_t)n * a.ntiles + tile];
      const float2 rq = a.ranges[(int64_t)(a.nb + np) * a.ntiles + tile];
      int K0, K1;
      range_window(rq.x - rk.y, rq.y - rk.x, a.e0, a.inv_de, a.ne, K0, K1);
      can = rk.x <= rk.y && rq.x <= rq.y && K0 <= K1 && crosses(rk.x, rk.y, rq.x, rq.y, a.ef) &&
            (region_possible(0, rk.x, rk.y, rq.x, rq.y, a.ef) || region_possible(1, rk.x, rk.y, rq.x, rq.y, a.ef));
    }
    for (uint64_t live = __ballot(can); live; live &= live - 1) {
      if (k++ % a.parts != part) continue;
      chi_unit<NORB, WT>(a, tile, n, n0 + __builtin_ctzll(live), sh);
      __syncthreads();
    }
  }
}

template <int NORB>
hipError_t launch_chi(const ChiArgs& a, ChiSplineArgs& c, int wtype, int grid, hipStream_t s) {
  const int64_t units = (int64_t)c.f.ntiles * c.nb * c.parts;
  for (c.first = 0; c.first < units; c.first += c.nunits) {
    c.nunits = (int)std::min<int64_t>(units - c.first, 1 << 22);  // a launch holds fewer than 2^32 work items
    c.per_xcd = (c.nunits + NXCD - 1) / NXCD;
    const hipError_t e = launch_chi_spline<NORB>(c, s);
    if (e != hipSuccess) return e;
  }
  if (wtype == TETRA_W_F16)
    hipLaunchKernelGGL((chi_kernel<NORB, _Float16>), dim3(grid), dim3(NT), 0, s, a);
  else if (wtype == TETRA_W_C32)
    hipLaunchKernelGGL((chi_kernel<NORB, float2>), dim3(grid), dim3(NT), 0, s, a);
  else
    hipLaunchKernelGGL((chi_kernel<NORB, float>), dim3(grid), dim3(NT), 0, s, a);
  return hipGetLastError();
}

}  // namespace

int64_t chi_units(const tetra_desc& d, int shape) {
  const TileShape sh = tile_shape(shape);
  const int64_t ntiles = (int64_t)((d.n1 + sh.x - 1) / sh.x) * ((d.n2 + sh.y - 1) / sh.y) * ((d.n3 + sh.z - 1) / sh.z);
  return ntiles * d.nb * d.nb;
}

int64_t chi_range_entries(const tetra_desc& d, int shape) {
  const TileShape sh = tile_shape(shape);
  return 2 * (int64_t)d.nb * ((d.n1 + sh.x - 1) / sh.x) * ((d.n2 + sh.y - 1) / sh.y) * ((d.n3 + sh.z - 1) / sh.z);
}

hipError_t chi(const tetra_desc& d, int q1, int q2, int q3, float e_fermi, const float* eps, const void* w, int wtype,
               const float* w_scale, float* out, int shape, void* ranges_ws, hipStream_t s) {
  ChiArgs a;
  a.eps = eps;
  a.w = w;
  a.w_scale = w_scale;
  a.out = out;
  a.n1 = d.n1;
  a.n2 = d.n2;
  a.n3 = d.n3;
  a.nb = d.nb;
  a.ne = d.ne;
  a.q1 = ((q1 % d.n1) + d.n1) % d.n1;
  a.q2 = ((q2 % d.n2) + d.n2) % d.n2;
  a.q3 = ((q3 % d.n3) + d.n3) % d.n3;
  a.ef = e_fermi;
  a.e0 = d.e0;
  a.de = d.de;
  a.inv_de = 1.0f / d.de;
  a.V = (float)(1.0 / (24.0 * (double)d.n1 * d.n2 * d.n3));
  const TileShape sh = tile_shape(shape);
  a.t1 = (d.n1 + sh.x - 1) / sh.x;
  a.t2 = (d.n2 + sh.y - 1) / sh.y;
  a.t3 = (d.n3 + sh.z - 1) / sh.z;
  // As many tiles as the shape gives, no longer than the grid needs: 24^3 x 12 x 12 x 300 (12 along axis 3 instead of
  // 16) 410 -> 394 us.
  a.TX = (d.n1 + a.t1 - 1) / a.t1;
  a.TY = (d.n2 + a.t2 - 1) / a.t2;
  a.TZ = (d.n3 + a.t3 - 1) / a.t3;
  a.ntiles = a.t1 * a.t2 * a.t3;
  // Workgroups per (tile, band n): more of them even out the pairs that do contribute, a few per (tile, n); each
  // takes its time to start, whether it finds a pair or not (10 ns for one of the spline pass). 64^3 x 8 x 8 x 500:
  // spline pass 0.82, 0.75, 0.71, 0.84, 0.98 ms for 1, 2, 3, 4, 8, clipping 0.89, 0.71, 0.83 ms for 1, 2, 4. Up to
  // one per pair on small grids.
  auto parts = [&](int64_t ntiles, int aim) {
    return (int)std::min<int64_t>(d.nb, std::max<int64_t>(1, aim / (ntiles * d.nb)));
  };
  a.parts = parts(a.ntiles, 16384);
  a.nunits = a.ntiles * d.nb * a.parts;
  a.per_xcd = (a.nunits + NXCD - 1) / NXCD;
  const int grid = a.per_xcd * NXCD;
  a.ranges = static_cast<const float2*>(ranges_ws);
  ChiSplineArgs c;
  c.f = forward_args(d, eps, w, wtype, w_scale, out, false);
  c.nb = d.nb;
  c.parts = parts(c.f.ntiles, 12288);
  c.q1 = a.q1;
  c.q2 = a.q2;
  c.q3 = a.q3;
  c.ef = e_fermi;
  c.ranges = a.ranges;
  c.TX = a.TX;
  c.TY = a.TY;
  c.TZ = a.TZ;
  c.u2 = a.t2;
  c.u3 = a.t3;
  c.ut = a.ntiles;
  hipError_t e = fill_zero(out, (int64_t)d.ne * d.norb, s);
  if (e != hipSuccess) return e;
  if (ranges_ws) {
    hipLaunchKernelGGL(chi_ranges_kernel, dim3(a.ntiles * d.nb), dim3(NT), 0, s, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  switch (d.norb) {
#define TETRA_CASE(N) \
  case N:             \
    return launch_chi<N>(a, c, wtype, grid, s);
    TETRA_CASE(1) TETRA_CASE(2) TETRA_CASE(3) TETRA_CASE(4) TETRA_CASE(5) TETRA_CASE(6) TETRA_CASE(7)
    TETRA_CASE(8) TETRA_CASE(9) TETRA_CASE(10) TETRA_CASE(11) TETRA_CASE(12) TETRA_CASE(13)
    TETRA_CASE(14) TETRA_CASE(15) TETRA_CASE(16)
#undef TETRA_CASE
    default:
      return hipErrorInvalidValue;
  }
}

}  // namespace tetra
