// Which of a launch's work-groups is the last to arrive, counted in memory that every one of them sees.  Host code too
// (any compiler), so that the counting can be tested without a device.
#pragma once

#include <cstddef>
#include <cstdint>

#ifdef __HIPCC__
#define SHELL_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define SHELL_HOST_DEVICE inline
#endif

namespace shell {

// Work-groups arrive in groups of 16, the last of a group at the root, because adds to one address pass one at a
// time: 512 work-groups that finish together spent 5 us on one counter, and spend 2 us on 33.
constexpr int kArriveGroup = 16, kArriveStride = 32;  // counters lie in cache lines of their own
SHELL_HOST_DEVICE constexpr size_t arrival_counters(long n) {
    return size_t(kArriveStride) * size_t(1 + (n + kArriveGroup - 1) / kArriveGroup);
}

// True for the last of the n work-groups.  wrap(counter, top) adds one, or sets a counter that stands at `top` to
// zero, and returns what it was, in one operation.  The counters (at zero before) so return to zero by the arrivals alone,
// also those of launches that share them and overlap: such launches spoil their own results and no later one's.  A
// reset apart from the last add could erase another launch's arrivals for good.
template <typename Wrap>
SHELL_HOST_DEVICE bool arrive_last(uint32_t* counters, long blk, long n, Wrap wrap) {
    const long g = blk / kArriveGroup, groups = (n + kArriveGroup - 1) / kArriveGroup;
    const long rest = n - g * kArriveGroup;
    const uint32_t top = uint32_t((rest < kArriveGroup ? rest : kArriveGroup) - 1), root = uint32_t(groups - 1);
    if (wrap(counters + kArriveStride * (1 + g), top) != top) return false;
    return groups == 1 || wrap(counters, root) == root;
}

}  // namespace shell
