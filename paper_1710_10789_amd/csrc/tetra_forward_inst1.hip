// Forward kernels for 1, 5, 9, 13 orbitals.
#include "tetra_forward_kernels.h"

namespace tetra {

#define TETRA_CASE(N)                                                       \
  template hipError_t launch_fwd<N>(const FwdArgs& a, int grid, hipStream_t s); \
  template hipError_t launch_batched<N>(const BatchArgs& b, int wtype, hipStream_t s);
TETRA_CASE(1) TETRA_CASE(5) TETRA_CASE(9) TETRA_CASE(13)
#undef TETRA_CASE

}  // namespace tetra
