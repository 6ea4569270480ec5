// rules.h -- the host's choices between the library's ways of doing the same work, as
// functions of sizes, types and flags alone (no HIP, so that a CPU test can ask them).
#ifndef LAZYTRAIN_RULES_H
#define LAZYTRAIN_RULES_H

#include <cstdint>

namespace rules {

// ----------------------------------------------------------- the norm's finish

// Waves that combine one tensor's chunk sums (1 or 4) and tensors per workgroup, for K
// tensors of which the longest has `longest` chunks.  A wave's round of loads covers 512
// chunks, four waves' 2048, so a few long tensors want four waves each.  The workgroups
// are counted at one address, some 40 ns for each, so a long list wants few of them.
// Norms of bf16 gradients in a captured graph, against a workgroup of four waves or four
// tensors at every length: nine tensors of 100M elements in all (longest 3500 chunks)
// 41.0 -> 39.5 us, 288 tensors of 20M 16.9 -> 15.7, the 3B-class model (325 tensors, an
// embedding of 38000 chunks) 890 -> 882.
constexpr int kFinishMany = 64;
struct FinishGeom {
    int waves, tensors;
};
constexpr FinishGeom finish_geom(int K, int64_t longest)
{
    if (K > kFinishMany)
        return longest > 4096 ? FinishGeom{4, 4} : FinishGeom{1, 16};
    return longest > 1024 ? FinishGeom{4, 1} : FinishGeom{1, 4};
}

// ------------------------------------------------------------------ 8-bit step

// What the choice of a step kernel for one launch depends on.
struct StepList {
    int B;               // block size
    bool dynamic;        // code map
    int64_t elems = 0;   // of all tensors
    int64_t blocks = 0;  // of all tensors, partial ones among them
    int64_t longest = 0; // elements of the longest block
};

inline StepList step_list(const int64_t* numels, int K, int B, bool dynamic)
{
    StepList l{B, dynamic};
    for (int k = 0; k < K; ++k) {
        l.elems += numels[k];
        l.blocks += (numels[k] + B - 1) / B;
        const int64_t block = numels[k] < B ? numels[k] : B;
        l.longest = block > l.longest ? block : l.longest;
    }
    return l;
}

// A step over much more data than the 256 MB Infinity Cache holds streams best with two
// workgroups per CU: further waves only mix more reads with writes in the memory system.
// Linear map, us a step, two per CU against the three or four that fit:
//   elements     48M            66M            96M            462M
//   B = 128     125.7, 123.8   178.5, 185.2   261.3, 273.1   1338, 1373
//   B = 1024    124.5, 124.5   176.7, 182.3   260.6, 270.3   1315, 1344
//   B = 4096    131.1, 124.1   179.8, 180.1   262.9, 267.1   1303, 1320
// (one per CU is 15% slower).  With the dynamic map at B = 8192 the kernel keeps the three
// that fit at every size: 368.0 us against 384.2 with two at 128M, 1324 against 1366 at
// 462M; at B = 2048 and 4096, with 16 elements per lane, it keeps three where an element
// moves 10 bytes and two where it moves 12 or more (fp32 gradients, a bf16 copy): B = 2048
// 553 us against 564 with two at 192M, with the copy 643 against 636, with fp32
// gradients 638 against 616; B = 4096 552 against 565, 642 against 634, 640 against 617.
// The elements count and not the kernel's work units: 13000
// tensors of 64 elements are a small step.
constexpr int64_t kStepStreamElems = 60 << 20;

// Workgroups per CU of the kernel for powers of two; 0: as many as fit.  `wide`: the
// gradients are fp32 or some tensor has a bf16 copy.
inline int step_per_cu(const StepList& l, bool wide)
{
    if (l.elems < kStepStreamElems || (l.dynamic && l.B == 8192))
        return 0;
    return l.dynamic && (l.B == 2048 || l.B == 4096) && !wide ? 3 : 2;
}

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
