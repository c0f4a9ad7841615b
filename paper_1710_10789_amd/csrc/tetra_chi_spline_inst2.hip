// The susceptibility's spline pass for 9 to 12 orbitals.
#include "tetra_chi_spline_kernels.h"

namespace tetra {

template hipError_t launch_chi_spline<9>(const ChiSplineArgs&, hipStream_t);
template hipError_t launch_chi_spline<10>(const ChiSplineArgs&, hipStream_t);
template hipError_t launch_chi_spline<11>(const ChiSplineArgs&, hipStream_t);
template hipError_t launch_chi_spline<12>(const ChiSplineArgs&, hipStream_t);

}  // namespace tetra
