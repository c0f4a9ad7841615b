// The susceptibility's spline pass for 13 to 16 orbitals.
#include "tetra_chi_spline_kernels.h"

namespace tetra {

template hipError_t launch_chi_spline<13>(const ChiSplineArgs&, hipStream_t);
template hipError_t launch_chi_spline<14>(const ChiSplineArgs&, hipStream_t);
template hipError_t launch_chi_spline<15>(const ChiSplineArgs&, hipStream_t);
template hipError_t launch_chi_spline<16>(const ChiSplineArgs&, hipStream_t);

}  // namespace tetra
