// Where the parts of a divided train range meet: two keys per query and a count of
// finished parts per query group.
//
// Parts run on any XCD, each with an L2 of its own.  All that they exchange goes through
// device-scope atomic accesses, which do not stop at an XCD's L2, so a part's wavefronts
// only wait for theirs (wait_device_accesses), meet at the workgroup's barrier and count
// the part: whoever then sees the count sees the minima, as atomic accesses of its own.
// Plain loads and stores would not be ordered by that, which is why the words are private
// to these classes: only clear() writes plainly, in a launch before the parts'.
// A release and an acquire at the count would order plain accesses as well, but a release
// writes the XCD's L2 back: by one wavefront per part, 63 pairs of 2754 rows took 156 us
// with it and 147 without, 30 of 5000 207 and 200, 8 of 12,000 276 and 265; by every
// wavefront, 47 uneven pairs around 5000 rows 390 and 331, one pair of 20,000 x 20,000
// 139 and 120.
#pragma once

#include "internal.h"

namespace latch {

// Waits until this wavefront's device-scope accesses have been performed.
__device__ __forceinline__ void wait_device_accesses() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// The two smallest keys (distance << 32 | index) that parts have brought.  With
// k1 <= k2 a part's best two, old = min(first, k1) as it was before and then
// min(second, min(k2, max(old, k1))): every k1 but the smallest is the larger of some
// such pair once, so `second` ends as the second smallest of all.
class PartKeys {
public:
    // Keys of query `at` of a slot.  (The arithmetic and the accesses are those of plain
    // words: on this type's own the FP4 kernel, which has no register to spare, compiles to
    // 1.5% to 3% more time.)
    static __device__ __forceinline__ PartKeys *of(PartKeys *slot, int at)
    {
        return reinterpret_cast<PartKeys *>(reinterpret_cast<uint64_t *>(slot) + 2 * at);
    }
    __device__ __forceinline__ void clear()
    {
        *reinterpret_cast<ulonglong2 *>(this) = make_ulonglong2(kNoNeighbour, kNoNeighbour);
    }
    __device__ __forceinline__ void merge(uint64_t k1, uint64_t k2)
    {
        auto *to = reinterpret_cast<unsigned long long *>(this);
        const uint64_t old = atomicMin(to, (unsigned long long)k1);
        atomicMin(to + 1, (unsigned long long)min(k2, max(old, k1)));
    }
    __device__ __forceinline__ uint64_t first() { return load(reinterpret_cast<uint64_t *>(this)); }
    __device__ __forceinline__ uint64_t second() { return load(reinterpret_cast<uint64_t *>(this) + 1); }

private:
    static __device__ __forceinline__ uint64_t load(uint64_t *p)
    {
        return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    [[maybe_unused]] uint64_t words_[2];
};
static_assert(sizeof(PartKeys) == 16, "a slot's size");

class PartCount {
public:
    __device__ __forceinline__ void clear() { *reinterpret_cast<uint32_t *>(this) = 0u; }
    // The count before this part.
    __device__ __forceinline__ uint32_t add_one() { return atomicAdd(reinterpret_cast<uint32_t *>(this), 1u); }

private:
    [[maybe_unused]] uint32_t n_;
};

}  // namespace latch
