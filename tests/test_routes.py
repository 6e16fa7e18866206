"""Host rules that choose between two ways of doing the same call."""
import itertools

import pytest

from . import routes


def test_ranges_overlap_as_sets_of_bytes():
    r = routes.load()
    for p, q in itertools.product(range(8), repeat=2):
        for pn, qn in itertools.product(range(5), repeat=2):
            want = bool(set(range(p, p + pn)) & set(range(q, q + qn)))
            assert bool(r.ranges_overlap(16 + p, pn, 16 + q, qn)) == want, (p, pn, q, qn)
    top = 2 ** 64 - 16
    assert r.ranges_overlap(top, 16, top + 15, 1) and not r.ranges_overlap(top, 15, top + 15, 1)


def test_a_kernel_writes_only_memory_of_the_one_device():
    """Memory, handle and current device: a handle of one device may not write a peer's memory by a kernel, whichever
    of the two is current, nor may a handle whose stream is another device's (-1)."""
    r = routes.load()
    for memory, handle, current in itertools.product((0, 1), (-1, 0, 1), (0, 1)):
        assert bool(r.one_device(memory, handle, current)) == (memory == handle == current)


# beams, groups, kernel, echo selection, range mode, groups held per CU, wave workgroups held per CU
@pytest.mark.parametrize("frame,waves", [
    ((32000, 16000, 11, 11, 0, 0, 4, 4), True),       # a pinhole camera's frame
    ((5000, 4688, 11, 11, 0, 0, 4, 4), True),         # a stateless frame
    ((9000, 9000, 13, 12, 2, 0, 8, 8), True),
    ((9000, 9000, 13, 12, 5, 0, 8, 8), True),
    ((2432, 2432, 11, 11, 0, 0, 8, 8), True),         # single beams
    ((3000, 3000, 9, 9, 0, 0, 7, 4), True),
    ((4129, 4129, 41, 3, 4, 0, 4, 4), True),
    ((8196, 4320, 7, 7, 0, 0, 8, 8), True),           # pairs
    ((13500, 7400, 9, 9, 0, 0, 7, 4), True),
    ((19500, 4920, 11, 11, 0, 0, 8, 8), True),        # full groups
    ((3000, 3000, 9, 9, 2, 2, 8, 8), True),           # range intervals, one pass
    ((9000, 7200, 11, 11, 0, 2, 8, 8), True),
    # each of these was slower by the wave (1.06 to 2.6 times)
    ((2300, 2300, 9, 9, 0, 2, 8, 8), False),
    ((6500, 5500, 13, 11, 0, 2, 8, 8), False),
    ((24000, 6600, 9, 9, 0, 2, 8, 8), False),
    ((9000, 9000, 15, 3, 0, 2, 8, 8), False),
    ((9000, 9000, 9, 9, 0, 1, 8, 8), False),          # corrected ranges have a kernel of their own
    ((1256, 1256, 9, 9, 4, 0, 8, 8), False),
    ((3900, 3250, 5, 5, 0, 0, 7, 4), False),
    ((26000, 6624, 9, 9, 4, 0, 8, 8), False),         # full groups, raw selection
    ((2048, 1978, 9, 7, 0, 0, 8, 8), False),          # few groups
    ((4000, 3478, 9, 7, 0, 0, 8, 8), False),
    ((4000, 1000, 9, 7, 0, 0, 8, 8), False),          # full groups
    ((24000, 6000, 9, 7, 0, 0, 4, 4), False),
    ((6504, 5636, 9, 7, 0, 0, 7, 4), False),          # many groups resident per CU (1200 bins)
    ((32000, 8000, 9, 7, 0, 0, 7, 4), False),
    ((8000, 6278, 1, 141, 0, 0, 4, 4), False),        # long kernels
    ((8000, 2897, 141, 1, 0, 0, 8, 8), False),
    ((8000, 5282, 21, 7, 0, 0, 4, 4), False),
    ((8000, 8000, 11, 11, 0, 2, 4, 4), False),        # range intervals
    ((17256, 17256, 9, 7, 1, 0, 8, 8), False),        # every run's key: strongest, longest
    ((17256, 17256, 9, 7, 3, 0, 8, 8), False),
    ((32000, 32000, 13, 13, 0, 0, 8, 8), False),      # more than 160 cells
    ((0, 0, 1, 1, 0, 0, 8, 8), False),
])
def test_frames_in_waves(frame, waves):
    assert routes.in_waves(*frame) == waves


@pytest.mark.parametrize("cells,corrected,lines", [
    (121, False, {8000: 8}), (160, False, {8000: 8}), (161, False, {1500: 4}), (1000, False, {1500: 4}),
    (1001, False, {400: 4, 1000: 8}), (144225, False, {400: 4, 1000: 8}), (25, True, {600: 8}), (144225, True, {600: 8})])
def test_bands_of_groups(cells, corrected, lines):
    """Every group goes to one XCD once; one band per XCD below the lines, several from them on."""
    for n in [*range(1, 70), 399, 400, 401, 599, 600, 999, 1000, 1001, 1499, 1500, 3330, 7199, 7999, 8000, 8031, 28800]:
        band, chunk = routes.xcd_share(n, cells, corrected)
        bands = max([1, *(b for line, b in lines.items() if n >= line)])
        assert band == -(-n // (8 * bands)) and chunk % band == 0 and chunk // band <= bands
        seen = sorted(g for x in range(8) for i in range(chunk) if (g := (i // band * 8 + x) * band + i % band) < n)
        assert seen == list(range(n)), n
