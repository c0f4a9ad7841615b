// Forward kernels for 4, 8, 12, 16 orbitals.
#include "tetra_forward_kernels.h"

namespace tetra {

#define TETRA_CASE(N)                                                       \
  template hipError_t launch_fwd<N>(const FwdArgs& a, int grid, hipStream_t s); \
  template hipError_t launch_batched<N>(const BatchArgs& b, int wtype, hipStream_t s);
TETRA_CASE(4) TETRA_CASE(8) TETRA_CASE(12) TETRA_CASE(16)
#undef TETRA_CASE

}  // namespace tetra
