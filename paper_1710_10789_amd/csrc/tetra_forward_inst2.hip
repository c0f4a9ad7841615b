// Forward kernels for 2, 6, 10, 14 orbitals.
#include "tetra_forward_kernels.h"

namespace tetra {

#define TETRA_CASE(N)                                                       \
  template hipError_t launch_fwd<N>(const FwdArgs& a, int grid, hipStream_t s); \
  template hipError_t launch_batched<N>(const BatchArgs& b, int wtype, hipStream_t s);
TETRA_CASE(2) TETRA_CASE(6) TETRA_CASE(10) TETRA_CASE(14)
#undef TETRA_CASE

}  // namespace tetra
