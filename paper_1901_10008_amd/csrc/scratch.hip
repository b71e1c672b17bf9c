// The scratch of sk_launch_static for plans whose device list needs more than a plan's table may (see LARGE_SCRATCH_BYTES).  A code object
// of its own: the runtime clears an array when it loads the object that holds it, 0.4 ms per MiB, which only a process that launches
// such a plan pays, once (25 ms at the first static launch of any plan when this was one array with the other).
#include <hip/hip_runtime.h>

#include "sk_internal.h"

static __device__ __align__(256) unsigned char large_scratch[sk::LARGE_SCRATCH_BYTES];

int sk::large_scratch_address(void **ptr) { return (int)hipGetSymbolAddress(ptr, HIP_SYMBOL(large_scratch)); }
