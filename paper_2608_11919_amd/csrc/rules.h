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

// The block sizes of k_adamw8_step: powers of two up to 8192.
constexpr bool is_power_block(int B) { return (B & (B - 1)) == 0 && B <= 8192; }

// What the choice of a step kernel for one launch depends on.
struct StepList {
    int B;                // block size
    bool dynamic;         // code map
    int64_t elems = 0;    // of all tensors
    int64_t blocks = 0;   // of all tensors, partial ones among them, and elements of the
    int64_t longest = 0;  // longest block: 0 at power blocks, whose rules do not ask (the
                          // divisions take 1.2 us for 288 tensors)
};

inline StepList step_list(const int64_t* numels, int K, int B, bool dynamic)
{
    StepList l{B, dynamic};
    for (int k = 0; k < K; ++k)
        l.elems += numels[k];
    if (is_power_block(B))
        return l;
    for (int k = 0; k < K; ++k) {
        l.blocks += (numels[k] + B - 1) / B;
        const int64_t block = numels[k] < B ? numels[k] : B;
        l.longest = block > l.longest ? block : l.longest;
    }
    return l;
}

// A step over much more data than the 256 MB Infinity Cache holds streams best with two
// workgroups per CU: further waves only mix more reads with writes in the memory system.
// Linear map, us a step, two per CU against the three or four that fit:
//   elements     44M            48M            54M            66M            92M
//   B = 128     112.9, 112.3   123.7, 123.9   148.5, 151.9   178.5, 185.2   261.3, 273.1
//   B = 1024    111.7, 110.8   123.3, 123.0   146.7, 148.7   176.7, 182.3   260.6, 270.3
//   B = 4096    119.3, 110.7   130.9, 122.9   148.6, 146.1   179.8, 180.1   262.9, 267.1
// and at 462M B = 128 1338, 1373, B = 1024 1315, 1344, B = 4096 1303, 1320
// (one per CU is 15% slower).  With the dynamic map at B = 8192 the kernel keeps the three
// that fit at every size: 368.0 us against 384.2 with two at 128M, 1324 against 1366 at
// 462M; at B = 2048 and 4096, with 16 elements per lane, it keeps three where an element
// moves 10 bytes and two where it moves 12 or more (fp32 gradients, a bf16 copy): B = 2048
// 553 us against 564 with two at 192M, with the copy 643 against 636, with fp32
// gradients 638 against 616; B = 4096 552 against 565, 642 against 634, 640 against 617.
// The elements count and not the kernel's work units: 13000
// tensors of 64 elements are a small step.
constexpr int64_t kStepStreamElems = 60 << 20;
constexpr int64_t kStepStreamElemsSmall = 50 << 20;  // linear map, B <= 1024

// Workgroups per CU of the kernel for powers of two; 0: as many as fit.  `wide`: the
// gradients are fp32 or some tensor has a bf16 copy.
inline int step_per_cu(const StepList& l, bool wide)
{
    const bool small = !l.dynamic && l.B <= 1024;
    if (l.elems < (small ? kStepStreamElemsSmall : kStepStreamElems) ||
        (l.dynamic && l.B == 8192))
        return 0;
    return l.dynamic && (l.B == 2048 || l.B == 4096) && !wide ? 3 : 2;
}

// Block sizes that are no power of two: waves that share a block, granules per lane and
// blocks per unit of k_adamw8_any, or waves = 0: k_adamw8_generic, 256 threads per block
// that read a block's gradients and codes twice.  Few granules per lane keep many waves in
// flight, which the dynamic map's table reads and small lists want; on large lists rows of
// busy lanes matter as much.  us a step, bf16 gradients (l: linear, d: dynamic map):
//
// * B <= 1024, up to three blocks per CU: a workgroup each.  {4, 1}, {1, 2} and {1, 4}: B = 768
//   l, 0.3M elements 5.5, 6.6, 8.2; B = 384 l, 0.2M 5.4, 6.4, 9.6; B = 448 d, 0.3M 7.1, 7.6.
//   Above that blocks queue: B = 448 l, 0.5M 7.2, 6.8.
// * B <= 1024, {1, 2} where it keeps 832 of a wave's 1024 elements busy, 704 with the
//   dynamic map or below 32M elements, and any number below 12M; else {1, 4}.  {1, 2} and
//   {1, 4}: B = 768 l 8M 29.3, 32.4; 32M 94.7, 95.5; 138M 412, 394.  B = 576 l 1M 8.4, 10.4;
//   8M 32.6, 34.4; 20M 73.4, 70.8; 92M 309, 279.  B = 704 d 1M 9.4, 10.4; 48M 162, 166.  B =
//   832 l 1M 8.2, 10.4; 32M 93, 108; 138M 415, 413.
// * B <= 8192: the fewest waves of two or three granules.  B = 1536 l, 138M (fp32 gradients)
//   562 with {4, 1}, 553 with {1, 4}, d 580, 612; B = 3072 552 with {4, 2}, 623 with {4, 4};
//   B = 5120 d 603 with {4, 3}, 624 with {8, 2}.  Where no block is longer than the 2048
//   elements the generic kernel takes in one go: 288 tensors of 0.1M elements in all, B =
//   8128 l 4.8 against 7.6 with {8, 2}; B = 5120 4.8, 7.5; B = 3072 4.8, 6.0.  With ten
//   thousand tensors {4, 2} is the better one again (B = 2112 l, 14M 81, 97).
// * B <= 16384, {16, 2}: a workgroup fills a CU.  Blocks that the generic kernel takes in
//   two goes (four, when the blocks are more than the CUs): 288 tensors of 0.1M 4.8
//   against 15.0, of 2M 13.7, 17.1, of 3M 22.6, 19.1 (B = 12288 l).  Below 14336 many lanes
//   are idle.  Generic and {16, 2}: B = 8256 l 2M 13.1, 16.5; 20M 67.2, 78.6; 92M 333, 319; B =
//   8256 d 1M 16.1, 11.2; 32M 100, 132; 138M 480, 510; B = 12288 d 4M 24.3, 21.9; 32M 101, 110;
//   92M 324, 291; B = 12288 l 30M 97, 108 (288 tensors); 48M 155, 147.
// * larger B: generic.
struct AnyGeom {
    int waves, granules, blocks;
};
constexpr int64_t kCus = 256;  // compute units of a gfx950 card
constexpr int kAnyMaxBlock = 16384;

inline AnyGeom any_geom(const StepList& l)
{
    constexpr AnyGeom generic = {0, 0, 1};
    const int B = l.B;
    if (B > kAnyMaxBlock)
        return generic;
    if (B > 8192) {
        if (l.longest <= (l.blocks > kCus ? 8192 : 4096))
            return generic;
        const bool large = l.elems >= (l.dynamic ? kStepStreamElems : int64_t(40) << 20);
        if (B < 12288 && l.blocks > kCus && (l.dynamic || !large))
            return generic;
        if (B >= 12288 && B < 14336 && l.blocks > 2 * kCus && !large)
            return generic;
        return {16, 2, 1};
    }
    if (B > 2048) {
        if (l.longest <= 2048 && (B > 4096 || l.blocks <= 16 * kCus))
            return generic;
        return B > 6144 ? AnyGeom{8, 2, 1} : AnyGeom{4, B <= 4096 ? 2 : 3, 1};
    }
    if (B > 1024 || l.blocks <= 3 * kCus)
        return {4, 1, 1};
    const int busy = 1024 / B * B;  // elements of {1, 2}'s 1024
    if (busy >= 832 || (busy >= 704 && (l.dynamic || l.elems < (32 << 20))) ||
        l.elems < (12 << 20))
        return {1, 2, 1024 / B};
    return {1, 4, 2048 / B};
}

// ------------------------------------------------------------- fp32-state step

// Workgroups per CU of the fp32-state step over `elems` elements; 0: as many as fit (four
// with bf16 gradients and no copy, else five).  Three stream best from some 24M elements
// on, most of all where four would fit (bf16 gradients, us a step, four and three): 20M
// 86.4, 86.4; 32M 174, 169; 64M 352, 342; 128M 713, 679; 330M 1825, 1745; 2.9e9 16690, 15360.
// Two are up to 10% slower there.  With five against three: 128M (fp32 gradients) 738,
// 736; 2.9e9 16680, 16550.
inline int step32_per_cu(int64_t elems) { return elems >= (24 << 20) ? 3 : 0; }

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
