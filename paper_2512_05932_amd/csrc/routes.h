// Host rules that choose between two ways of doing the same call: plain C++
// without HIP, so that tests can compile them by themselves.
#pragma once

#include <cstddef>
#include <cstdint>

#include "../../include/lidar_sim.h"

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

// Whether a single frame whose groups hold up to four beams runs with a wave per
// group (which takes the group's beams one after another) instead of a
// workgroup per group.  A beam takes the wave longer, and the frame as long as
// its fullest groups, so there have to be enough groups to fill the chip: the
// more, the more beams share a group (their pixels are read once for all there)
// and the more groups a CU holds.  `held` per CU of the group kernel (by its
// LDS), `held_wave` per CU of the wave kernel (eight with one pass).
//
// The lines lie where the last frames that lose end, over 289 frames of 1200 to
// 20000 beams in grids, Lissajous figures and jittered grids on a road and on
// i.i.d. surfaces (512, 1200 and 2048 bins) and 2520 frames of 1200 to 60000
// beams in runs of one, two and four, on these and on a flat wall, with and
// without sun, kept waveforms and raw selection.  Against the groups the first
// take 0.91 of the time on average (0.99 with every frame of 2048 beams in waves,
// 2.2 at most there) and 1.04 at most, the second 0.80 and 1.17 at most; 2432
// single beams of an 11 x 11 kernel 33.1 and 25.7 us.  What loses is shared groups
// on i.i.d. surfaces with 2048 bins, where every pixel ends a run: at random places
// 0.92 to 1.35 (kept waveforms), where the road takes 0.62 to 0.90 and the wall 0.59
// to 0.83.  Left to the groups, with their times (groups, waves):
//  * few groups: 2048 beams of a 9 x 7 kernel in 1978 groups 24.6 and 36.9 us;
//  * full groups: 24000 beams of a 9 x 7 kernel in 6000 groups (2048 bins) 1.09 of
//    the time; raw selections, whose waveforms are not convolved, 0.74 to 1.40
//    with 7000 full groups;
//  * 513 to some 1600 bins, where a CU holds more groups: 6504 beams of a 9 x 7
//    kernel in 5636 groups, 1200 bins, 40.9 and 47.9 us;
//  * long kernels, whose rows or columns the wave walks alone: 4000 beams of a
//    1 x 141 kernel 38.5 and 51.1 us; kernels of more than 160 cells: 4000 beams
//    of 400 samples 36 and 46 us;
//  * range intervals with more than 512 bins, a step per bin of a pixel's range: 8000
//    beams of an 11 x 11 kernel 93 and 240 us (2048 bins).  With one pass they are
//    as centre ranges, whatever the bins' width (2268 frames): single beams gain
//    from 2500 groups on (0.31 to 0.87 of the time from 3300 on), beams that share
//    groups from 6500 on (0.41 to 1.12), full groups lose up to 1.7;
//  * selections that need every run's key, which are not found as the waveform
//    is written: 17256 beams of 64 samples, strongest echo, 92 and 98 us.
struct FrameShape {
    long beams, groups;
    int kernel_w, kernel_h;
    uint32_t select, range_mode;    // LIDAR_ECHO_*, LIDAR_RANGE_*
    int held, held_wave;
};

constexpr long kNarrowCells = 160;

inline bool frame_in_waves(const FrameShape& f)
{
    constexpr int kRound = 13, kLong = 41;
    if (f.select == LIDAR_ECHO_STRONGEST || f.select == LIDAR_ECHO_LONGEST) return false;
    if ((f.range_mode != LIDAR_RANGE_CENTRE && f.range_mode != LIDAR_RANGE_INTERVAL) || f.groups <= 0) return false;
    const int extent = f.kernel_w > f.kernel_h ? f.kernel_w : f.kernel_h;
    if ((long)f.kernel_w * f.kernel_h > kNarrowCells || extent > kLong) return false;
    const double per_group = (double)f.beams / (double)f.groups;
    if (f.select >= LIDAR_ECHO_RAW_STRONGEST && per_group > 2.5) return false;
    const bool shared = per_group > 1.01, one_pass = f.held_wave >= 8;
    double need = 2000.0;                                            // single beams
    if (f.range_mode == LIDAR_RANGE_INTERVAL) {
        if (!one_pass || per_group > 2.5 || extent > kRound) return false;
        need = shared ? 6500.0 : 2500.0;
    } else if (shared) {
        if (one_pass) need = 3450.0 + 330.0 * per_group;
        else if (f.held > f.held_wave) need = 5000.0 + 900.0 * per_group;
        else need = 3500.0 + 1000.0 * per_group;
        if (extent > kRound) need += 2000.0;
    }
    return (double)f.groups >= need;
}

// Bands of consecutive groups that an XCD takes of a frame.  Groups are in
// column order, so one band per XCD keeps the most pixels in its L2, but columns
// differ in cost, and workgroups go to the XCDs in turn, whatever these have
// left.  Times in us with 1, 2, 4 and 8 bands: 28800 beams of 83000 samples 932,
// 831, 756, 772 (the mean of six scenes 760 and 765 with 4 and 8, but 833 and 824
// on the benchmark's); 14400 beams of 21000 corrected samples, which read less for
// their FP64 arithmetic, 888, 796, 779, 750 (another scene 1010, 796, 727, 729);
// 32000 beams of 105 samples (in waves) 137, 136, 133, 131.  Over 300 frames of 25
// to 100000 cells and 200 to 20000 beams on a road and on i.i.d. surfaces:
//  * corrected ranges: 8 bands take 0.90 of the time with one from 1000 groups on
//    (0.82 to 1.00), 0.98 with 600 to 1000, and 4 bands 0.91;
//  * more than 1000 cells: 8 bands take 0.95 from 1000 groups on (0.75 to 1.10), as 4
//    do; with 400 to 1000 groups 4 take 0.99 (0.93 to 1.05) and 8 take 1.01;
//  * 161 to 1000 cells: 4 bands take 0.97 from 1500 groups on (0.89 to 1.02),
//    1.00 with 1000 to 1500 (0.92 to 1.10);
//  * up to 160 cells: within 0.02 of each other, except for large frames on a
//    road, above.
inline int xcd_bands(long groups, long cells, bool corrected)
{
    if (corrected) return groups < 600 ? 1 : 8;
    if (cells <= kNarrowCells) return groups < 8000 ? 1 : 8;
    if (cells <= 1000) return groups < 1500 ? 1 : 4;
    return groups < 400 ? 1 : groups < 1000 ? 4 : 8;
}

// Groups of a band, and of an XCD's bands together (its last ones may lie past
// the frame's groups).
struct XcdShare {
    int band, chunk;
};

inline XcdShare xcd_share(int groups, long cells, bool corrected, int xcds)
{
    const int bands = xcd_bands(groups, cells, corrected);
    const int band = groups > 0 ? (groups - 1) / (xcds * bands) + 1 : 1;
    return {band, groups > 0 ? ((groups - 1) / (xcds * band) + 1) * band : 0};
}

}  // namespace lidar
