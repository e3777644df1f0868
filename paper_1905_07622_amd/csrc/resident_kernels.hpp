// Selection of the resident kernel instantiations.
#pragma once

#include "resident.hpp"

namespace femheat {

template <typename V, int KIND>
const void* resident_kernel_planes(int planes) {
  switch (planes) {
    case 3: return reinterpret_cast<const void*>(&resident_kernel<V, KIND, 3>);
    case 5: return reinterpret_cast<const void*>(&resident_kernel<V, KIND, 5>);
    case 9: return reinterpret_cast<const void*>(&resident_kernel<V, KIND, 9>);
    default: return nullptr;
  }
}

template <typename V>
const void* resident_kernel_of(int kind, int planes) {
  return kind == kElemCubic  ? resident_kernel_planes<V, kElemCubic>(planes)
         : kind == kElemTet6 ? resident_kernel_planes<V, kElemTet6>(planes)
                             : resident_kernel_planes<V, kElemBox>(planes);
}

}  // namespace femheat
