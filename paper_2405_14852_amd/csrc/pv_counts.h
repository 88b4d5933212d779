// What the blocks of a call count (groups decided, codes changed), without a launch that clears it, which alone lasts
// 4.7 us: a context has two sets of words and its calls take turns.  Every word that a call finds was cleared by the
// call before it, and its first kernel clears the other set for the one after it; so what a call leaves in its own
// does not matter to the next.  A captured call is replayed when and where the caller likes, so it keeps off these
// two: it has a third set, behind a launch that clears it.  Two levels of words, a cache line each: atomics on one
// address are served one after the other, about 10 ns each.  One context's calls are ordered by its stream.
#pragma once
#include <hip/hip_runtime.h>

constexpr int kCountSlots = 32, kCountStride = 16;
constexpr int kCountFast = (kCountSlots + 1) * kCountStride;     // three words of the beam filter's
constexpr int kCountList = kCountFast + kCountStride, kCountChanged = kCountList + kCountStride;
constexpr int kCountWords = kCountChanged + kCountStride;
constexpr size_t kCountBytes = (size_t)kCountWords * 8;

// `mine` is zero when a call's first kernel starts, which clears `next`, if there is one (pv_counts_clear).
// pv_counters gives them out.
struct pv_counts {
    unsigned long long *mine = nullptr, *next = nullptr;
};

#ifdef __HIPCC__
// All threads (at least kCountWords / kCountStride) of every block of a call's first kernel.
__device__ __forceinline__ void pv_counts_clear(const pv_counts &c)
{
    if (c.next && blockIdx.x == 0 && threadIdx.x < kCountWords / kCountStride) c.next[threadIdx.x * kCountStride] = 0ull;
}

// One thread of each of the `blocks` blocks that count calls this once.  a < 2^40 over all of them, blocks < 2^24.
// True in the last one: *total is the sum.
__device__ __forceinline__ bool pv_counts_arrive(unsigned long long *words, unsigned blocks, unsigned long long a,
                                                 unsigned long long *total)
{
    constexpr unsigned long long kOne = 1ull << 40;
    unsigned arrivals = blocks;
    if (blocks > (unsigned)kCountSlots) {
        const unsigned slot = blockIdx.x % kCountSlots;
        a += kOne;
        a += atomicAdd(words + slot * kCountStride, a);
        if ((unsigned)(a >> 40) != (blocks - slot + kCountSlots - 1) / kCountSlots) return false;
        a &= kOne - 1ull;
        arrivals = kCountSlots;
    }
    a += kOne;
    a += atomicAdd(words + kCountSlots * kCountStride, a);
    if ((unsigned)(a >> 40) != arrivals) return false;
    *total = a & (kOne - 1ull);
    return true;
}

// A group that the beam filter leaves to the exact kernel; the list has room for the call's k groups.
__device__ __forceinline__ void pv_list_redo(const pv_counts &c, int32_t *list, int64_t k, int n)
{
    const unsigned long long slot = atomicAdd(c.mine + kCountList, 1ull);
    if (slot < (unsigned long long)k) list[slot] = n;
}
#endif
