// Forward pass: host side (kernels in tetra_forward_kernels.h, instantiated per orbital count in
// tetra_forward_inst*.hip).

#include <algorithm>
#include <cmath>

#include "tetra_forward_args.h"
#include "tetra_spline.h"

namespace tetra {

namespace {

constexpr int NXCD = 8;

__global__ void fill_zero_kernel(float* p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0.0f;
}

// Exact-mode set-up: no bound yet, every accumulator at zero (plain stores: capturable in a graph).
__global__ void exact_init_kernel(int* gexp, unsigned long long* acc, int64_t n) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *gexp = kNoBound;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    acc[i] = 0ull;
}
}  // namespace

constexpr int kSide = 8;  // largest tile side, in cubes
constexpr int kCus = 256;

FwdArgs forward_args(const tetra_desc& d, const float* eps, const void* w, int wtype, const float* w_scale, float* dos,
                     bool alone) {
  FwdArgs a;
  a.eps = eps;
  a.w = w;
  a.w_scale = w_scale;
  a.dos = dos;
  a.gexp = nullptr;
  a.gacc = nullptr;
  a.wtype = wtype;
  a.n1 = d.n1;
  a.n2 = d.n2;
  a.n3 = d.n3;
  a.ne = d.ne;
  a.e0 = d.e0;
  a.de = d.de;
  a.inv_de = 1.0f / d.de;
  a.e0d = d.e0;
  a.ded = d.de;
  a.ned = d.ne;
  const double V = 1.0 / (24.0 * (double)d.n1 * d.n2 * d.n3);  // V_T / (4 V_G)
  a.V = (float)V;
  a.inv_ded = 1.0 / (double)d.de;
  a.c4 = 4.0 * V * a.inv_ded;
  // The errors of the tetrahedra next to the limit average over the tetrahedra of an energy: the limit falls
  // with their number (from 16^3 points x 8 bands on, to a tenth at 32 times that), by the power that keeps
  // the error of the sum (error of one ~ limit^-3/4, number^-1/2). 64^3 x 8 x 8 x 1000: 0.174 against
  // 0.184 ms with the same error, 3.0e-7, against FP64; a hundredth would raise it to 4.2e-7.
  const double points = (double)d.n1 * d.n2 * d.n3 * d.nb;
  a.unit = step_unit(d.de);
  a.width = d.de * a.unit;
  const float width4 = a.width * a.width * a.width * a.width;
  a.degenerate = kDegenerate / (float)std::min(10.0, std::max(1.0, std::pow(points / 32768.0, 2.0 / 3.0))) * width4;
  a.degenerate_exact = kDegenerateExact * width4;
  a.window = false;
  a.joff = 0.0;
  a.Vd = V;
  a.out_scale = 1.0;
  a.shift = 0;
  const int n[3] = {d.n1, d.n2, d.n3};
  // Tiles of 8 x 8 x 8 whatever shape the caller asks for: with the sides of the shapes the forward took 0.29 ms
  // (8 x 8 x 4) to 0.63 ms (4 x 8 x 4) at 64^3 x 8 x 8 x 1000 against 0.17 ms. Where these leave half of the CUs or more
  // without a workgroup, tiles of half or a quarter of that, at the same number of lanes: a unit's time is what counts
  // there. 16^3 x 8 x 8 x 100 22 -> 18 us, four simple cubic bands 54 -> 23 us (42 us before the spline form).
  int side[3] = {kSide, kSide, kSide};
  auto tiles = [&](int i) { return (n[i] + side[i] - 1) / side[i]; };
  for (int i = 0; alone && i < 2 && 2ll * tiles(0) * tiles(1) * tiles(2) * d.nb <= kCus; ++i) side[i] = kSide / 2;
  int t[3], s[3], r[3], lanes = 1;
  for (int i = 0; i < 3; ++i) {
    t[i] = tiles(i);
    s[i] = n[i] / t[i];
    r[i] = n[i] % t[i];
    lanes *= s[i] + (r[i] > 0);
  }
  a.lanes = std::max((lanes + 63) / 64 * 64, side[0] < kSide ? 512 : 256);  // small tiles: more lanes than cubes
  a.t2 = t[1];
  a.t3 = t[2];
  a.s1 = s[0];
  a.s2 = s[1];
  a.s3 = s[2];
  a.r1 = r[0];
  a.r2 = r[1];
  a.r3 = r[2];
  a.ntiles = t[0] * t[1] * t[2];
  a.nunits = a.ntiles * d.nb;
  a.by_ntiles = fast_div(a.ntiles);
  a.by_t2 = fast_div(a.t2);
  a.by_t3 = fast_div(a.t3);
  a.per_xcd = (a.nunits + NXCD - 1) / NXCD;
  a.lg_units = 0;
  while ((1ll << a.lg_units) < (long long)a.nunits) ++a.lg_units;
  return a;
}

namespace {

// Whether the loop over every tetrahedron's window is the faster one. Its time grows with the energies of a window,
// about ne / n of them on a grid of n points a side, the spline form's does not; the exact mode runs the spline form
// twice and pays for its bound. The windows of an energy grid over a part of the bands are longer, so the lines lie
// where the loop still is no slower over a third of them. Spline form -> loop, ms, whole bands (a third of them):
//   64^3 x 8 x 8 x 32 0.163 -> 0.156 (0.166 -> 0.186), x 16 x 32 0.270 -> 0.211; 96^3 x 8 x 8 x 64 0.509 -> 0.490
//   exact 64^3 x 8 x 8 x 64 0.335 -> 0.266, x 128 0.326 -> 0.291 (0.295 -> 0.315), x 256 0.315 -> 0.326;
//   96^3 x 8 x 8 x 128 1.034 -> 0.862 (0.941 -> 0.862), 32^3 x 8 x 8 x 32 0.060 -> 0.050 (x 48 0.055 -> 0.069)
// On a grid with one point along two axes every tetrahedron has equal energies: 1 x 1 x 4096 x 4 x 8 0.040 -> 0.025.
bool few_energies(const tetra_desc& d, bool exact) {
  if ((d.n1 == 1) + (d.n2 == 1) + (d.n3 == 1) > 1) return true;
  const double face = std::cbrt((double)d.n1 * d.n2 * d.n3) * std::cbrt((double)d.n1 * d.n2 * d.n3);
  return (exact ? (d.norb > 8 ? 55.0 : 40.0) : d.norb > 8 ? 110.0 : 200.0) * d.ne <= face;
}

// The arguments of tetra_window_kernels.h.
FwdArgs window_args(FwdArgs a, const tetra_desc& d) {
  const TileShape sh = tile_shape(0);
  a.window = true;
  a.s1 = sh.x;
  a.s2 = sh.y;
  a.s3 = sh.z;
  a.t2 = (d.n2 + sh.y - 1) / sh.y;
  a.t3 = (d.n3 + sh.z - 1) / sh.z;
  a.ntiles = (d.n1 + sh.x - 1) / sh.x * a.t2 * a.t3;
  a.nunits = a.ntiles * d.nb;
  a.per_xcd = (a.nunits + NXCD - 1) / NXCD;
  a.lg_units = 0;
  while ((1ll << a.lg_units) < (long long)a.nunits) ++a.lg_units;
  return a;
}

}  // namespace

hipError_t fill_zero(float* p, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t blocks = std::min<int64_t>((n + 255) / 256, 4096);
  hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)blocks), dim3(256), 0, s, p, n);
  return hipGetLastError();
}

hipError_t forward(const tetra_desc& d, const float* eps, const void* w, int wtype, const float* w_scale, float* dos,
                   void* exact_scratch, hipStream_t s) {
  FwdArgs a = forward_args(d, eps, w, wtype, w_scale, dos, true);
  if (few_energies(d, exact_scratch != nullptr)) a = window_args(a, d);
  // exact_scratch (exact mode): 256 bytes holding the largest bound exponent, then ne*norb 64-bit sums
  a.gexp = exact_scratch ? static_cast<int*>(exact_scratch) : nullptr;
  a.gacc = exact_scratch ? reinterpret_cast<unsigned long long*>(static_cast<char*>(exact_scratch) + 256) : nullptr;
  const int grid = a.per_xcd * NXCD;
  hipError_t e = hipSuccess;
  if (exact_scratch) {
    const int64_t n = (int64_t)d.ne * d.norb;
    hipLaunchKernelGGL(exact_init_kernel, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 4096)), dim3(256), 0, s,
                       a.gexp, a.gacc, n);
    e = hipGetLastError();
  } else {
    e = fill_zero(dos, (int64_t)d.ne * d.norb, s);
  }
  if (e != hipSuccess) return e;
  switch (d.norb) {
#define TETRA_CASE(N) \
  case N:             \
    return launch_fwd<N>(a, grid, s);
    TETRA_CASE(1) TETRA_CASE(2) TETRA_CASE(3) TETRA_CASE(4) TETRA_CASE(5) TETRA_CASE(6) TETRA_CASE(7)
    TETRA_CASE(8) TETRA_CASE(9) TETRA_CASE(10) TETRA_CASE(11) TETRA_CASE(12) TETRA_CASE(13)
    TETRA_CASE(14) TETRA_CASE(15) TETRA_CASE(16)
#undef TETRA_CASE
    default:
      return hipErrorInvalidValue;
  }
}

size_t batched_launches(const tetra_item* items, int n) {
  size_t launches = 0;
  for (int norb = 1; norb <= 16; ++norb) {
    int cnt = 0;
    for (int i = 0; i < n; ++i) cnt += items[i].d.norb == norb;
    launches += (cnt + kMaxBatch - 1) / kMaxBatch;
  }
  return launches;
}

hipError_t batched(const tetra_item* items, int n, int wtype, hipStream_t s) {
  for (int norb = 1; norb <= 16; ++norb) {
    BatchArgs b;
    b.n = 0;
    b.total = 0;
    b.lanes = 64;
    for (int i = 0; i <= n; ++i) {
      const bool flush = (i == n && b.n > 0) || b.n == kMaxBatch;
      if (flush) {
        b.per_xcd = (b.total + NXCD - 1) / NXCD;
        hipError_t e = hipSuccess;
        switch (norb) {
#define TETRA_CASE(N) \
  case N:             \
    e = launch_batched<N>(b, wtype, s); \
    break;
          TETRA_CASE(1) TETRA_CASE(2) TETRA_CASE(3) TETRA_CASE(4) TETRA_CASE(5) TETRA_CASE(6) TETRA_CASE(7)
          TETRA_CASE(8) TETRA_CASE(9) TETRA_CASE(10) TETRA_CASE(11) TETRA_CASE(12) TETRA_CASE(13)
          TETRA_CASE(14) TETRA_CASE(15) TETRA_CASE(16)
#undef TETRA_CASE
          default:
            e = hipErrorInvalidValue;
        }
        if (e != hipSuccess) return e;
        b.n = 0;
        b.total = 0;
        b.lanes = 64;
      }
      if (i == n) break;
      const tetra_desc& d = items[i].d;
      if (d.norb != norb) continue;
      BatchItem& it = b.it[b.n++];
      const FwdArgs f = forward_args(d, items[i].eps, items[i].w, wtype, nullptr, items[i].dos, n == 1);
      it.eps = items[i].eps;
      it.w = items[i].w;
      it.w_scale = wtype == TETRA_W_F16 ? items[i].w_scale : nullptr;
      it.dos = items[i].dos;
      it.n1 = d.n1;
      it.n2 = d.n2;
      it.n3 = d.n3;
      it.ne = d.ne;
      it.e0 = d.e0;
      it.de = d.de;
      it.t2 = f.t2;
      it.t3 = f.t3;
      it.s = f.s1 | f.s2 << 8 | f.s3 << 16;
      it.r1 = f.r1;
      it.r2 = f.r2;
      it.r3 = f.r3;
      it.by_ntiles = f.by_ntiles;
      it.by_t2 = f.by_t2;
      it.by_t3 = f.by_t3;
      it.ntiles = f.ntiles;
      it.degenerate = f.degenerate;
      it.unit_begin = b.total;
      b.total += f.nunits;
      b.lanes = std::max(b.lanes, f.lanes);
    }
  }
  return hipSuccess;
}

}  // namespace tetra
