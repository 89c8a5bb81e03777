// Kernel arguments read in place (device code of the .hip files).
#pragma once
#include <hip/hip_runtime.h>

namespace stitch {

// The kernel's first argument (a descriptor, or an array of them) where the launch put it, in the
// constant address space: uniform reads of it are scalar loads, at any index.  (The parameter's
// own address is that of a private copy, which only an optimizing build does without.)
template <typename D>
__device__ __forceinline__ const __attribute__((address_space(4))) D* first_arg() {
  return (const __attribute__((address_space(4))) D*)__builtin_amdgcn_kernarg_segment_ptr();
}

}  // namespace stitch
