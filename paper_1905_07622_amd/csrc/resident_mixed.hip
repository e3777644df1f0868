// Resident kernels of the mixed form (see resident.hpp) for every element
// kind and brick height; one file per form, so that they build side by side.
#include "resident_kernels.hpp"

namespace femheat {

const void* resident_kernel_mixed(int kind, int planes) { return resident_kernel_of<float, false>(kind, planes); }

}  // namespace femheat
