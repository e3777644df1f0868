// Selection of the resident kernel instantiations.
#pragma once

#include "resident.hpp"

namespace femheat {

template <typename V, int KIND, bool CHEB>
const void* resident_kernel_planes(int planes) {
  switch (planes) {
    case 3: return reinterpret_cast<const void*>(&resident_kernel<V, KIND, 3, CHEB>);
    case 5: return reinterpret_cast<const void*>(&resident_kernel<V, KIND, 5, CHEB>);
    case 9: return reinterpret_cast<const void*>(&resident_kernel<V, KIND, 9, CHEB>);
    default: return nullptr;
  }
}

template <typename V, bool CHEB>
const void* resident_kernel_of(int kind, int planes) {
  if (kind == kElemCubic) return resident_kernel_planes<V, kElemCubic, CHEB>(planes);
  if (kind == kElemTet6) {
    if constexpr (CHEB)  // (tetrahedra run with the Jacobi preconditioner)
      return nullptr;
    else
      return resident_kernel_planes<V, kElemTet6, CHEB>(planes);
  }
  return resident_kernel_planes<V, kElemBox, CHEB>(planes);
}

}  // namespace femheat
