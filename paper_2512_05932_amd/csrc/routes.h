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

// Whether a kernel on the handle's stream may write memory of device `memory`
// in place of the copy engine, which reaches every device: only where that
// memory, the handle (its arrays and its stream; -1: these differ) and the
// current device are one.
inline bool one_device(int memory, int handle, int current)
{
    return handle >= 0 && memory == handle && current == handle;
}

}  // namespace lidar
