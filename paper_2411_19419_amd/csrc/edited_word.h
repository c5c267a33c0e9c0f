// The note that column-compressed arrays do not hold what the build wrote (csc_gather_kernel.h, apply_kernels.h).
#pragma once
#include <hip/hip_runtime.h>

namespace convspmv {

// A word of the device that one plan has to itself.  It holds `stamp` from the first product on that found the arrays
// edited (before, another value, whatever an earlier plan left there).
struct EditedWord {
    unsigned *word;
    unsigned stamp;
};
__device__ __forceinline__ bool noted_edited(const EditedWord &e) { return *const_cast<const volatile unsigned *>(e.word) == e.stamp; }

}  // namespace convspmv
