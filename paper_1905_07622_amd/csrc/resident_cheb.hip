// Resident kernels of the FP64 form with the Chebyshev preconditioner (see
// resident.hpp) for hexahedra and every brick height; one file per form,
// so that they build side by side.
#include "resident_kernels.hpp"

namespace femheat {

const void* resident_kernel_cheb(int kind, int planes) { return resident_kernel_of<double, true>(kind, planes); }

}  // namespace femheat
