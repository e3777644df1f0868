// Validation of coefficient arrays where they are (checks.hip).
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

namespace femheat {

struct CoefficientArrays {
  const double *k, *rhoc;
  size_t n;
};

// Bit 0 of bad[i]: some k of arrays[i] is negative or not finite; bit 1: some
// rho*c is not positive or not finite.  False where an array is not plain
// device memory of `device` over its whole length (a caller's mistake, or
// memory of another kind) or a HIP call fails: the caller then copies the
// arrays to the host and checks them there.
bool check_coefficients_on_device(const CoefficientArrays* arrays, int32_t n, int device, int32_t* bad);

}  // namespace femheat
