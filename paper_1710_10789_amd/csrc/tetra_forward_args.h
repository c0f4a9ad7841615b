// Launch arguments of the forward kernels (tetra_forward_kernels.h), shared by the host side
// (tetra_forward.hip) and the files that instantiate the kernels per orbital count.
#pragma once

#include "tetra_internal.h"

namespace tetra {

constexpr int kNoBound = -100000;  // *gexp before any workgroup has a bound

// Division of a 31-bit number by a constant: (n m) >> s.
struct FastDiv {
  uint32_t m;
  int s;
};
inline FastDiv fast_div(int d) {
  int l = 0;
  while ((1ll << l) < d) ++l;
  return {(uint32_t)(((1ull << (31 + l)) + d - 1) / d), 31 + l};
}

struct FwdArgs {
  const float* eps;
  const void* w;         // float, _Float16 or float2 (complex amplitude) [nb][norb][nk]
  const float* w_scale;  // per-band scale of _Float16 weights
  float* dos;
  int* gexp;                 // exact mode: largest bound exponent of any workgroup (atomicMax in mode 1)
  unsigned long long* gacc;  // exact mode: [ne][norb] sums in the common 64-bit fixed point (mode 2)
  int lg_units;              // exact mode: ceil(log2(nunits))
  int wtype;                 // TETRA_W_* of w
  int n1, n2, n3, ne;
  float e0, de, inv_de, V;
  float unit, width;   // a power of two and a grid step in energies times it (tetra_spline.h)
  float degenerate;    // limit of a degenerate tetrahedron (tetra_spline.h) in these, times rows^3
  float degenerate_exact;  // the same of the exact mode
  double e0d, ded, ned;  // e0, de and ne in FP64 (from the arguments straight into scalar registers)
  double inv_ded, c4;    // 1/de and 4 V_T/(4 V_G) / de in FP64
  int t2, t3;          // tiles along axes 2 and 3
  int s1, s2, s3;      // cubes of the smaller tiles along each axis; the first r1, r2, r3 have one more
  int r1, r2, r3;
  FastDiv by_ntiles, by_t2, by_t3;
  int ntiles, nunits, per_xcd;
  int lanes;    // workgroup size: a lane per cube of the largest tile, in whole waves
  bool window;  // tetra_window_kernels.h with tiles of s1 x s2 x s3 cubes (the last ones partly outside the grid)
  // number of states: grid index j stands for e0 + (j + joff) de and goes to output row j - shift (rows below
  // 0 are dropped), times out_scale; Vd = V_T/(4 V_G)
  double joff, Vd, out_scale;
  int shift;
};

// Problems of a batched launch (items in order, units band-major): what differs between them, small
// enough for 32 of them to travel as kernel arguments.
struct BatchItem {
  const float* eps;
  const void* w;
  const float* w_scale;
  float* dos;
  int n1, n2, n3, ne;
  float e0, de;
  int t2, t3;
  int s;  // s1, s2, s3, a byte each
  int r1, r2, r3;
  FastDiv by_ntiles, by_t2, by_t3;
  int ntiles;
  float degenerate;
  int unit_begin;  // first global unit of this item
};

struct BatchArgs {
  int n, total, per_xcd;
  int lanes;  // workgroup size: of the problem with the largest tiles
  BatchItem it[kMaxBatch];
};
static_assert(sizeof(BatchArgs) <= 4096, "kernel arguments");

// The arguments that do not depend on the kind of sum; alone: there are no other problems to fill the chip with.
FwdArgs forward_args(const tetra_desc& d, const float* eps, const void* w, int wtype, const float* w_scale, float* dos,
                     bool alone);

// Defined per orbital count in tetra_forward_inst*.hip.
template <int NORB>
hipError_t launch_fwd(const FwdArgs& a, int grid, hipStream_t s);
template <int NORB>
hipError_t launch_batched(const BatchArgs& b, int wtype, hipStream_t s);
template <int NORB>
hipError_t launch_nos(const FwdArgs& a, int grid, hipStream_t s);

}  // namespace tetra
