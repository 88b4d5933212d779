// What the blocks of a call count (groups decided, codes changed), without a launch that clears it: the
// words are zero between calls, the last block to arrive has the sums and leaves them zero again.  A
// launch that only clears lasts 4.7 us.  Two levels of words, a cache line each: atomics on one address
// are served one after the other, about 10 ns each.  One context's calls are ordered by its stream.
#pragma once
#include <hip/hip_runtime.h>

constexpr int kCountSlots = 32, kCountStride = 16;
constexpr int kCountFast = (kCountSlots + 1) * kCountStride;     // three words of the beam filter's
constexpr int kCountList = kCountFast + kCountStride, kCountChanged = kCountList + kCountStride;
constexpr int kCountWords = kCountChanged + kCountStride;
constexpr size_t kCountBytes = (size_t)kCountWords * 8;

#ifdef __HIPCC__
// One thread of each of the `blocks` blocks that count calls this once.  a < 2^40 over all of them, blocks < 2^24.
// True in the last one: *total is the sum.
__device__ __forceinline__ bool pv_counts_arrive(unsigned long long *words, unsigned blocks, unsigned long long a,
                                                 unsigned long long *total)
{
    constexpr unsigned long long kOne = 1ull << 40;
    unsigned long long *root = words + kCountSlots * kCountStride;
    unsigned arrivals = blocks;
    if (blocks > (unsigned)kCountSlots) {
        const unsigned slot = blockIdx.x % kCountSlots;
        a += kOne;
        a += atomicAdd(words + slot * kCountStride, a);
        if ((unsigned)(a >> 40) != (blocks - slot + kCountSlots - 1) / kCountSlots) return false;
        atomicExch(words + slot * kCountStride, 0ull);
        a &= kOne - 1ull;
        arrivals = kCountSlots;
    }
    a += kOne;
    a += atomicAdd(root, a);
    if ((unsigned)(a >> 40) != arrivals) return false;
    atomicExch(root, 0ull);
    *total = a & (kOne - 1ull);
    return true;
}
#endif
