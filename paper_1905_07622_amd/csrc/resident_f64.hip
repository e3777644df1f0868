// Resident kernels of the FP64 form (see resident.hpp) for every element
// kind and brick height (one file per form, so that they build side by
// side), and the kernel that prepares a launch of either.
#include "resident_host.hpp"
#include "resident_kernels.hpp"

namespace femheat {

const void* resident_kernel_f64(int kind, int planes) { return resident_kernel_of<double, false>(kind, planes); }

hipError_t resident_reset(hipStream_t stream, const ResSim* sims, uint32_t n, ResForm form, uint32_t max_nodes) {
  hipLaunchKernelGGL(resident_reset_kernel, resident_reset_grid(n, max_nodes), dim3(256), 0, stream, sims, n,
                     form == RES_MIXED ? 1 : 0);
  return hipGetLastError();
}

}  // namespace femheat
