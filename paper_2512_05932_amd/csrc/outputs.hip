// Results into the caller's device arrays: the echoes, counts, waveforms and
// beam records of a frame in one launch.
//
// A copy of its own per array costs a launch each, which a small frame (40 KB
// of results) pays as much as its footprint kernel: three copies of a
// 1000-beam frame took 8 us of the stream (4.8 us each once the clock is up),
// this kernel 4.0 us.  Large results are bound by HBM.
#include "engine.h"

namespace lidar {

namespace {

constexpr int kThreads = 256;
constexpr int kUnits = 4;                     // units of a thread

// Block b copies units of the segment whose blocks include b.
template <typename T>
__device__ inline void copy_units(const OutSegment& s, long block)
{
    const long n = s.bytes / (long)sizeof(T);
    const T* src = (const T*)s.src;
    T* dst = (T*)s.dst;
#pragma unroll
    for (int i = 0; i < kUnits; ++i) {
        const long u = (block * kUnits + i) * kThreads + threadIdx.x;
        if (u < n) *gptr(dst + u) = *gptr(src + u);
    }
}

__global__ __launch_bounds__(kThreads)
void k_copy_out(OutSegments a)
{
    long b = blockIdx.x;
    for (int i = 0; i < kOutSegments; ++i) {
        const OutSegment s = a.seg[i];
        if (b < s.blocks) {
            if (s.unit == 16) copy_units<gint4>(s, b);
            else if (s.unit == 8) copy_units<gint2>(s, b);
            else copy_units<int>(s, b);
            return;
        }
        b -= s.blocks;
    }
}

}  // namespace

bool out_segment(OutSegment* s, void* dst, const void* src, size_t bytes)
{
    const size_t low = (size_t)dst | (size_t)src | bytes;
    if (low % 4 != 0) return false;
    s->src = src;
    s->dst = dst;
    s->bytes = (long)bytes;
    // the widest unit that the addresses and the size allow (frames of a
    // batch lie at multiples of 8 and 4 bytes)
    s->unit = low % 16 == 0 ? 16 : low % 8 == 0 ? 8 : 4;
    const long per_block = (long)s->unit * kUnits * kThreads;
    s->blocks = (s->bytes + per_block - 1) / per_block;
    return true;
}

hipError_t launch_copy_out(hipStream_t s, const OutSegments& a)
{
    long blocks = 0;
    for (const OutSegment& g : a.seg) blocks += g.blocks;
    if (blocks == 0) return hipSuccess;
    if (blocks >= (1l << 31)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_copy_out, dim3((unsigned)blocks), dim3(kThreads), 0, s, a);
    return hipGetLastError();
}

}  // namespace lidar
