// Launch arguments of the susceptibility's spline pass (tetra_chi_spline_kernels.h), shared by the host side
// (tetra_chi.hip) and the files that instantiate the kernel per orbital count.
#pragma once

#include "tetra_forward_args.h"

namespace tetra {

struct ChiSplineArgs {
  FwdArgs f;  // the grid, the energies and the tiles; dos is the susceptibility's output
  int nb, parts;  // bands, workgroups per (tile, band n)
  int q1, q2, q3;  // transfer in grid steps, reduced to [0, n)
  float ef;
  // Energy ranges by (band, tile of a table of tiles of TX x TY x TZ cubes), u2 and u3 of them along axes 2 and
  // 3 and ut in all: rows [0, nb) at the tile's points, rows [nb, 2 nb) at the points shifted by q; or NULL.
  const float2* ranges;
  int TX, TY, TZ, u2, u3, ut;
  int64_t first;  // first of the nunits units (tile, band n, part) of this launch
  int nunits, per_xcd;
};

template <int NORB>
hipError_t launch_chi_spline(const ChiSplineArgs& a, hipStream_t s);

}  // namespace tetra
