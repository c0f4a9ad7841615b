// Number of states and bin-averaged DOS: host side (kernels in tetra_nos_kernels.h, instantiated per orbital
// count in tetra_nos_inst*.hip) and the sum over the energies.

#include <algorithm>

#include "tetra_forward_args.h"

namespace tetra {

namespace {

constexpr int NXCD = 8;

// In-place running sum over rows of p[n][norb], one workgroup per column, accumulated in FP64.
__global__ __launch_bounds__(256) void column_scan_kernel(float* p, int n, int norb) {
  __shared__ double s_part[256];
  const int m = blockIdx.x;
  const int tid = threadIdx.x;
  const int per = (n + 255) / 256;
  const int r0 = min(tid * per, n), r1 = min(r0 + per, n);
  double acc = 0.0;
  for (int r = r0; r < r1; ++r) acc += (double)p[(int64_t)r * norb + m];
  s_part[tid] = acc;
  __syncthreads();
  if (tid == 0) {
    double run = 0.0;
    for (int i = 0; i < 256; ++i) {
      const double v = s_part[i];
      s_part[i] = run;
      run += v;
    }
  }
  __syncthreads();
  double run = s_part[tid];
  for (int r = r0; r < r1; ++r) {
    run += (double)p[(int64_t)r * norb + m];
    p[(int64_t)r * norb + m] = (float)run;
  }
}

}  // namespace

hipError_t nos(const tetra_desc& d, const float* eps, const void* w, int wtype, const float* w_scale, float* out,
               bool binned, hipStream_t s) {
  FwdArgs a = forward_args(d, eps, w, wtype, w_scale, out, true);
  if (binned) {  // increments between the midpoints E_j -+ de/2: ne + 1 grid indices, the first dropped
    a.ne = d.ne + 1;
    a.ned = a.ne;
    a.joff = -0.5;
    a.shift = 1;
    a.out_scale = 1.0 / (double)d.de;
  }
  const int grid = a.per_xcd * NXCD;
  hipError_t e = fill_zero(out, (int64_t)d.ne * d.norb, s);
  if (e != hipSuccess) return e;
  switch (d.norb) {
#define TETRA_CASE(N)              \
  case N:                          \
    e = launch_nos<N>(a, grid, s); \
    break;
    TETRA_CASE(1) TETRA_CASE(2) TETRA_CASE(3) TETRA_CASE(4) TETRA_CASE(5) TETRA_CASE(6) TETRA_CASE(7)
    TETRA_CASE(8) TETRA_CASE(9) TETRA_CASE(10) TETRA_CASE(11) TETRA_CASE(12) TETRA_CASE(13)
    TETRA_CASE(14) TETRA_CASE(15) TETRA_CASE(16)
#undef TETRA_CASE
    default:
      return hipErrorInvalidValue;
  }
  if (e != hipSuccess || binned) return e;
  hipLaunchKernelGGL(column_scan_kernel, dim3(d.norb), dim3(256), 0, s, out, d.ne, d.norb);
  return hipGetLastError();
}

}  // namespace tetra
