// Number-of-states kernels for 1, 3, 5, 7, 9, 11, 13, 15 orbitals.
#include "tetra_nos_kernels.h"

namespace tetra {

#define TETRA_CASE(N) template hipError_t launch_nos<N>(const FwdArgs& a, int grid, hipStream_t s);
TETRA_CASE(1) TETRA_CASE(3) TETRA_CASE(5) TETRA_CASE(7) TETRA_CASE(9) TETRA_CASE(11) TETRA_CASE(13) TETRA_CASE(15)
#undef TETRA_CASE

}  // namespace tetra
