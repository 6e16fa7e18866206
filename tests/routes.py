"""The engine's host rules (csrc/routes.h), compiled by themselves as plain C++ for the tests."""
import ctypes as C
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = """
#include "routes.h"
extern "C" {
int ranges_overlap(const void* p, size_t pn, const void* q, size_t qn) { return lidar::ranges_overlap(p, pn, q, qn); }
int one_device(int memory, int handle, int current) { return lidar::one_device(memory, handle, current); }
int xcd_share(int groups, long cells, int corrected, int* chunk)
{
    const lidar::XcdShare s = lidar::xcd_share(groups, cells, corrected != 0, 8);
    *chunk = s.chunk;
    return s.band;
}
int in_waves(long beams, long groups, int kw, int kh, unsigned select, unsigned range_mode, int held, int held_wave)
{
    return lidar::frame_in_waves(lidar::FrameShape{beams, groups, kw, kh, select, range_mode, held, held_wave});
}
}
"""

_lib = None


def load():
    global _lib
    if _lib is None:
        with tempfile.TemporaryDirectory() as d:
            src, so = os.path.join(d, "rules.cpp"), os.path.join(d, "librules.so")
            with open(src, "w") as f:
                f.write(SOURCE)
            inc = [os.path.join(ROOT, "paper_2512_05932_amd", "csrc"), os.path.join(ROOT, "include")]
            subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", *[f"-I{i}" for i in inc], src, "-o", so],
                           check=True)
            _lib = C.CDLL(so)
        _lib.in_waves.argtypes = [C.c_long, C.c_long, C.c_int, C.c_int, C.c_uint, C.c_uint, C.c_int, C.c_int]
        _lib.xcd_share.argtypes = [C.c_int, C.c_long, C.c_int, C.POINTER(C.c_int)]
        _lib.ranges_overlap.argtypes = [C.c_void_p, C.c_size_t, C.c_void_p, C.c_size_t]
    return _lib


def in_waves(beams, groups, kernel_w, kernel_h, select, range_mode, held, held_wave) -> bool:
    return bool(load().in_waves(beams, groups, kernel_w, kernel_h, select, range_mode, held, held_wave))


def xcd_share(groups, cells, corrected=False):
    """Groups of a band and of an XCD."""
    chunk = C.c_int()
    return load().xcd_share(groups, cells, corrected, C.byref(chunk)), chunk.value
