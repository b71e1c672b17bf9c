// The kernels, in units of compilation (-DSK_UNIT=0 to 6): in one they take the compiler three minutes, side by side one.
#include <hip/hip_runtime.h>

#include "kernels.hip.h"

namespace sk {

// element type (-1: mixed), any alignment, narrow
#define SK_KERNEL(dt, any, narrow) template __global__ void sk_superkernel<dt, any, narrow>(const TileWork *__restrict__, KernelArgs);
#if SK_UNIT == 0
SK_KERNEL(SK_F32, false, true)
SK_KERNEL(SK_BF16, false, true)
SK_KERNEL(SK_F16, false, true)
SK_KERNEL(SK_F32, false, false)
#elif SK_UNIT == 1
SK_KERNEL(SK_BF16, false, false)
SK_KERNEL(SK_F16, false, false)
#elif SK_UNIT == 2
SK_KERNEL(SK_F32, true, false)
#elif SK_UNIT == 3
SK_KERNEL(SK_BF16, true, false)
#elif SK_UNIT == 4
SK_KERNEL(SK_F16, true, false)
#elif SK_UNIT == 5
SK_KERNEL(-1, false, false)
#elif SK_UNIT == 6
SK_KERNEL(-1, true, false)
#else
#error "SK_UNIT is 0 to 6"
#endif

}  // namespace sk
