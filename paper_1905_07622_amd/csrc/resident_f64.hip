// Resident kernels of the FP64 form (see resident.hpp) for every element
// kind and brick height (one file per form, so that they build side by
// side), and the kernel that prepares a launch of either.
#include <algorithm>

#include "resident_host.hpp"
#include "resident_kernels.hpp"

namespace femheat {

const void* resident_kernel_f64(int kind, int planes) { return resident_kernel_of<double, false>(kind, planes); }

hipError_t resident_reset(hipStream_t stream, const ResSim* sims, uint32_t n, ResForm form, uint32_t max_nodes) {
  const uint32_t x = std::max<uint32_t>(1, std::min<uint32_t>((max_nodes + 255) / 256, std::max<uint32_t>(8, 2048 / n)));
  hipLaunchKernelGGL(resident_reset_kernel, dim3(x, n), dim3(256), 0, stream, sims, form == RES_MIXED ? 1 : 0);
  return hipGetLastError();
}

}  // namespace femheat
