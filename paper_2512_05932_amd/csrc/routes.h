// Host rules that choose between two ways of doing the same call: plain C++
// without HIP, so that tests can compile them by themselves.
#pragma once

#include <cstddef>
#include <cstdint>

namespace lidar {

// Whether [p, p + pn) and [q, q + qn) share a byte.
inline bool ranges_overlap(const void* p, size_t pn, const void* q, size_t qn)
{
    const uintptr_t a = (uintptr_t)p, b = (uintptr_t)q;
    return pn > 0 && qn > 0 && (a <= b ? b - a < pn : a - b < qn);
}

}  // namespace lidar
