// The susceptibility's spline pass for 1 to 8 orbitals.
#include "tetra_chi_spline_kernels.h"

namespace tetra {

template hipError_t launch_chi_spline<1>(const ChiSplineArgs&, hipStream_t);
template hipError_t launch_chi_spline<2>(const ChiSplineArgs&, hipStream_t);
template hipError_t launch_chi_spline<3>(const ChiSplineArgs&, hipStream_t);
template hipError_t launch_chi_spline<4>(const ChiSplineArgs&, hipStream_t);
template hipError_t launch_chi_spline<5>(const ChiSplineArgs&, hipStream_t);
template hipError_t launch_chi_spline<6>(const ChiSplineArgs&, hipStream_t);
template hipError_t launch_chi_spline<7>(const ChiSplineArgs&, hipStream_t);
template hipError_t launch_chi_spline<8>(const ChiSplineArgs&, hipStream_t);

}  // namespace tetra
