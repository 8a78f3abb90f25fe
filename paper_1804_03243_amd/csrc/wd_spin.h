// Arithmetic of the waits in a cluster of workgroups, apart from the waits
// themselves so that it can be checked on the host.
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define WD_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define WD_HOST_DEVICE inline
#endif

namespace wd {

// Whether a count of arrivals has come to `target`.  The count goes on over a
// whole launch, modulo 2^32 (254 epsilon levels of 32 workgroups are 16 thousand
// arrivals a frame); it is never 2^31 away from a target that is waited for.
WD_HOST_DEVICE bool arrived(uint32_t now, uint32_t target) { return (int32_t)(now - target) >= 0; }

}  // namespace wd
