// The check of spline_check.cpp with the smallest limit that the kernels use (forward_args divides kDegenerate by up to
// ten for large problems). Test harness only: compiled by tests/test_spline_edges_host.py.
#include "tetra_forward_args.h"
#include "tetra_spline.h"

#define kDegenerate (kDegenerate / 10.0f)
#include "spline_check.cpp"
