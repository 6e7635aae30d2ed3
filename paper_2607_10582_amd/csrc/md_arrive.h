// A count of arrivals shared by the workgroups of one launch, by which the
// last of n of them finds out that it is the last.  Nobody waits: a caller
// arrives when its reads are done, and exactly one caller, whichever comes
// last, is told to do what may only be done after all of them.  The count is
// zero again before that caller goes on, so a launch leaves nothing behind
// for the next one, however late any workgroup was.
// (Compiled for the device and, for its test, for the host.)
#pragma once

#if defined(__HIP__)
#define MD_HD __attribute__((host, device, always_inline)) inline
#else
#define MD_HD inline
#endif

namespace md {

// Arrivals before this one.  On the device the caller's reads have returned
// (s_waitcnt vmcnt(0) and a barrier of its workgroup) when it arrives.
MD_HD int arrive(int* count) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __hip_atomic_fetch_add(count, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#else
    return __atomic_fetch_add(count, 1, __ATOMIC_ACQ_REL);
#endif
}

// Whether the caller that found `before` arrivals is the last of n; its
// count then starts again (every other caller has arrived, and does not
// touch it any more).
MD_HD bool arrive_last(int* count, int before, int n) {
    if (before != n - 1) return false;
    *count = 0;
    return true;
}

}  // namespace md
