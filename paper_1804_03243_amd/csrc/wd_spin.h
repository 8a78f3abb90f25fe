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

constexpr uint64_t kSpinTicks = 200000000; // a wait that has run this long (2 s of the 100 MHz clock) is an error, not a hang
constexpr uint64_t kSpinGap = 1000;        // longest time between two looks at the clock that counts (10 µs)
constexpr uint32_t kSpinLooks = 8;         // looks at the arrivals (about 0.7 µs each) for one at the clock

// Whether a count of arrivals has come to `target`.  The count goes on over a
// whole launch, modulo 2^32 (254 epsilon levels of 32 workgroups are 16 thousand
// arrivals a frame); it is never 2^31 away from a target that is waited for.
WD_HOST_DEVICE bool arrived(uint32_t now, uint32_t target) { return (int32_t)(now - target) >= 0; }

// The time a wait has been running.  A workgroup's queue may be descheduled
// while it waits: that time passes between two looks at the clock and does not
// count, nobody can arrive in it.
struct SpinClock {
  uint64_t last, spent;
  WD_HOST_DEVICE explicit SpinClock(uint64_t now) : last(now), spent(0) {}
  // Whether the wait has run beyond its limit, as of a look at `now`.
  WD_HOST_DEVICE bool beyond(uint64_t now) {
    const uint64_t gap = now - last;
    last = now;
    spent += gap < kSpinGap ? gap : kSpinGap;
    return spent > kSpinTicks;
  }
};

}  // namespace wd
