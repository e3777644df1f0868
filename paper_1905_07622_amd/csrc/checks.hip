// Validation of coefficient arrays in device memory (gfx950): k_e >= 0 and
// rho*c_e > 0, both finite, read where they are.  Copying them to the host for
// it took 17 of the 90 ms of a batch of 64 simulations of 49^3 nodes (2 x 0.9
// MB each, through pageable memory); the kernels take well under one.
#include <hip/hip_runtime.h>

#include <cmath>

#include "checks.hpp"

namespace femheat {
namespace {

// bit 0: some k is negative or not finite; bit 1: some rho*c is not positive or not finite
__global__ void __launch_bounds__(256) check_coefficients_kernel(const double* __restrict__ k,
                                                                 const double* __restrict__ rhoc, size_t n,
                                                                 int32_t* __restrict__ flag) {
  int bad = 0;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const double a = k[i], b = rhoc[i];
    if (!(a >= 0.0) || !isfinite(a)) bad |= 1;
    if (!(b > 0.0) || !isfinite(b)) bad |= 2;
  }
  if (bad) atomicOr(flag, bad);
}

__global__ void clear_flags_kernel(int32_t* flags, int32_t n) {
  for (int32_t i = threadIdx.x; i < n; i += blockDim.x) flags[i] = 0;
}

// Whether n doubles at p lie in one allocation of device `device`.
bool on_device(const double* p, size_t n, int device) {
  hipPointerAttribute_t a{};
  if (hipPointerGetAttributes(&a, p) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  if (a.type != hipMemoryTypeDevice || a.device != device) return false;
  hipDeviceptr_t base = nullptr;
  size_t size = 0;
  if (hipMemGetAddressRange(&base, &size, const_cast<double*>(p)) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  const char *b = static_cast<const char*>(base), *q = reinterpret_cast<const char*>(p);
  return q >= b && (reinterpret_cast<uintptr_t>(p) & 7u) == 0 && n * sizeof(double) <= size - (size_t)(q - b);
}

}  // namespace

// On the default stream, as the copies it replaces: after whatever a blocking
// stream of the caller's has been given.  The flags are allocated and freed in
// that stream's order too: hipFree waits for every stream of the device, so
// that a handle created beside a run of 400 ms took 404 ms instead of 5.
bool check_coefficients_on_device(const CoefficientArrays* arrays, int32_t n, int device, int32_t* bad) {
  for (int32_t i = 0; i < n; ++i)
    if (!on_device(arrays[i].k, arrays[i].n, device) || !on_device(arrays[i].rhoc, arrays[i].n, device)) return false;
  int32_t* flags = nullptr;
  if (hipMallocAsync(reinterpret_cast<void**>(&flags), (size_t)n * sizeof(int32_t), nullptr) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  hipLaunchKernelGGL(clear_flags_kernel, dim3(1), dim3(256), 0, nullptr, flags, n);
  for (int32_t i = 0; i < n; ++i) {
    const size_t blocks = std::min<size_t>((arrays[i].n + 1023) / 1024, 1024);
    hipLaunchKernelGGL(check_coefficients_kernel, dim3((uint32_t)blocks), dim3(256), 0, nullptr, arrays[i].k,
                       arrays[i].rhoc, arrays[i].n, flags + i);
  }
  bool ok = hipGetLastError() == hipSuccess;
  ok = hipMemcpy(bad, flags, (size_t)n * sizeof(int32_t), hipMemcpyDeviceToHost) == hipSuccess && ok;
  if (!ok) (void)hipGetLastError();
  (void)hipFreeAsync(flags, nullptr);
  return ok;
}

}  // namespace femheat
