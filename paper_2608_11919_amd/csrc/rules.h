// rules.h -- the host's choices between the library's ways of doing the same work, as
// functions of sizes, types and flags alone (no HIP, so that a CPU test can ask them).
#ifndef LAZYTRAIN_RULES_H
#define LAZYTRAIN_RULES_H

namespace rules {

// ------------------------------------------------- streamed step: pinned memory

// Flags of a pinned allocation (hipHostMalloc).
constexpr unsigned kHostDefault = 0x0, kHostCoherent = 0x40000000, kHostNonCoherent = 0x80000000;

// Whether the copy kernel may move arrays of a pinned allocation made with these flags.
// The GPU does not cache memory of the default and the coherent kind, so the kernel's
// plain loads and stores need no cache invalidated or written back between the host's
// accesses, other kernels' and the copy engines'.  Any other kind takes copy commands,
// which do not depend on it.
constexpr bool copy_kernel_takes(unsigned flags)
{
    return flags == kHostDefault ||
           ((flags & kHostCoherent) != 0 && (flags & kHostNonCoherent) == 0);
}

}  // namespace rules

#endif
