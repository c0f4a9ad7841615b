// Forward kernels for 3, 7, 11, 15 orbitals.
#include "tetra_forward_kernels.h"

namespace tetra {

#define TETRA_CASE(N)                                                       \
  template hipError_t launch_fwd<N>(const FwdArgs& a, int grid, hipStream_t s); \
  template hipError_t launch_batched<N>(const BatchArgs& b, int wtype, hipStream_t s);
TETRA_CASE(3) TETRA_CASE(7) TETRA_CASE(11) TETRA_CASE(15)
#undef TETRA_CASE

}  // namespace tetra
