// Number-of-states kernels for 2, 4, 6, 8, 10, 12, 14, 16 orbitals.
#include "tetra_nos_kernels.h"

namespace tetra {

#define TETRA_CASE(N) template hipError_t launch_nos<N>(const FwdArgs& a, int grid, hipStream_t s);
TETRA_CASE(2) TETRA_CASE(4) TETRA_CASE(6) TETRA_CASE(8) TETRA_CASE(10) TETRA_CASE(12) TETRA_CASE(14) TETRA_CASE(16)
#undef TETRA_CASE

}  // namespace tetra
